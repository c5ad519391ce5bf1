// The Wilson-Dirac stencil (Sec. 2.1, Eq. 1 and Eq. 2) for gfx950.
//
// One lane per output site (the paper's one-thread-per-site gather, no
// inter-lane communication).  Per direction the neighbour spinor is projected
// onto the two-spin half spinor of (1 -+ gamma_mu), the link (decoded from
// 18/12/8 stored reals in registers) multiplies the two colour vectors, and
// the lower spin components are rebuilt by the fixed spin map of the chiral
// representation.  Accumulation is in registers; the epilogue forms
//
//   t   = G5? [ a * self + b * (H in) ]
//   out = c0 * t + c1 * v1 + c2 * v2 + c3 * v3        (c_k may be device scalars)
//
// and optionally adds |out|^2 (FP64) into per-block partial sums.
// Chiral basis: gamma_mu = [[0, A_mu], [A_mu^H, 0]], A_0 = -1, A_k = -i sigma_k,
// so (1 - gamma_mu) psi = (h, -A^H h) with h = psi_up - A psi_dn, and
// (1 + gamma_mu) psi = (g, A^H g) with g = psi_up + A psi_dn.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "wilson.h"

using namespace ndq;

namespace {

// spin s, colour c -> component index 3*s + c; S: HopSpinor<R> or HopSpinor16
template <int MU, typename R, typename S>
__device__ __forceinline__ void hop_fwd(const S& s, const C<R> u[3][3], C<R> acc[12]) {
    C<R> h0[3], h1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (MU == 0) {
            h0[c] = s.add(c, 6 + c);
            h1[c] = s.add(3 + c, 9 + c);
        } else if constexpr (MU == 1) {
            h0[c] = s.addi(c, 9 + c);
            h1[c] = s.addi(3 + c, 6 + c);
        } else if constexpr (MU == 2) {
            h0[c] = s.add(c, 9 + c);
            h1[c] = s.sub(3 + c, 6 + c);
        } else {
            h0[c] = s.addi(c, 6 + c);
            h1[c] = s.subi(3 + c, 9 + c);
        }
    }
    C<R> w0[3], w1[3];
    const auto wt = s.weight();
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        w0[r] = cmul(u[r][0], h0[0]);
        w1[r] = cmul(u[r][0], h1[0]);
        w0[r] = cfma(w0[r], u[r][1], h0[1]);
        w1[r] = cfma(w1[r], u[r][1], h1[1]);
        w0[r] = cfma(w0[r], u[r][2], h0[2]);
        w1[r] = cfma(w1[r], u[r][2], h1[2]);
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        acc[r] = wt.acc(acc[r], w0[r]);
        acc[3 + r] = wt.acc(acc[3 + r], w1[r]);
        if constexpr (MU == 0) {
            acc[6 + r] = wt.acc(acc[6 + r], w0[r]);
            acc[9 + r] = wt.acc(acc[9 + r], w1[r]);
        } else if constexpr (MU == 1) {
            acc[6 + r] = wt.acc(acc[6 + r], cmulmi(w1[r]));
            acc[9 + r] = wt.acc(acc[9 + r], cmulmi(w0[r]));
        } else if constexpr (MU == 2) {
            acc[6 + r] = wt.acc(acc[6 + r], cneg(w1[r]));
            acc[9 + r] = wt.acc(acc[9 + r], w0[r]);
        } else {
            acc[6 + r] = wt.acc(acc[6 + r], cmulmi(w0[r]));
            acc[9 + r] = wt.acc(acc[9 + r], cmuli(w1[r]));
        }
    }
}

template <int MU, typename R, typename S>
__device__ __forceinline__ void hop_bwd_mul(const S& s, const C<R> u[3][3], C<R> w0[3], C<R> w1[3]) {
    C<R> g0[3], g1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (MU == 0) {
            g0[c] = s.sub(c, 6 + c);
            g1[c] = s.sub(3 + c, 9 + c);
        } else if constexpr (MU == 1) {
            g0[c] = s.subi(c, 9 + c);
            g1[c] = s.subi(3 + c, 6 + c);
        } else if constexpr (MU == 2) {
            g0[c] = s.sub(c, 9 + c);
            g1[c] = s.add(3 + c, 6 + c);
        } else {
            g0[c] = s.subi(c, 6 + c);
            g1[c] = s.addi(3 + c, 9 + c);
        }
    }
    // w = U^H g
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        w0[r] = cmulc(u[0][r], g0[0]);
        w1[r] = cmulc(u[0][r], g1[0]);
        w0[r] = cfmac(w0[r], u[1][r], g0[1]);
        w1[r] = cfmac(w1[r], u[1][r], g1[1]);
        w0[r] = cfmac(w0[r], u[2][r], g0[2]);
        w1[r] = cfmac(w1[r], u[2][r], g1[2]);
    }
}

template <int MU, typename R, typename W>
__device__ __forceinline__ void hop_bwd_acc(const W& s, const C<R> w0[3], const C<R> w1[3], C<R> acc[12]) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        acc[r] = s.acc(acc[r], w0[r]);
        acc[3 + r] = s.acc(acc[3 + r], w1[r]);
        if constexpr (MU == 0) {
            acc[6 + r] = s.acc(acc[6 + r], cneg(w0[r]));
            acc[9 + r] = s.acc(acc[9 + r], cneg(w1[r]));
        } else if constexpr (MU == 1) {
            acc[6 + r] = s.acc(acc[6 + r], cmuli(w1[r]));
            acc[9 + r] = s.acc(acc[9 + r], cmuli(w0[r]));
        } else if constexpr (MU == 2) {
            acc[6 + r] = s.acc(acc[6 + r], w1[r]);
            acc[9 + r] = s.acc(acc[9 + r], cneg(w0[r]));
        } else {
            acc[6 + r] = s.acc(acc[6 + r], cmuli(w0[r]));
            acc[9 + r] = s.acc(acc[9 + r], cmulmi(w1[r]));
        }
    }
}

template <int MU, typename R, typename S>
__device__ __forceinline__ void hop_bwd(const S& s, const C<R> u[3][3], C<R> acc[12]) {
    C<R> w0[3], w1[3];
    hop_bwd_mul<MU>(s, u, w0, w1);
    hop_bwd_acc<MU>(s.weight(), w0, w1, acc);
}

// PAIR64: FP64 also issues both hops' loads together (the direction split with
// 12- or 8-real links; 18-real ones would take the registers of a wavefront).
// `more` issues further loads behind those of the hops, before their arithmetic.
template <int SP, int LP, int RECON, int MU, bool NT, bool PAIR64, typename More>
__device__ __forceinline__ void hop_pair(const WilsonArgs& a, int p, int32_t i, const int32_t nb[8],
                                         const SpinorView& vin, C<typename SpinorIO<SP>::R> acc[12],
                                         More more) {
    using R = typename SpinorIO<SP>::R;
    using F = LinkFmt<LP, RECON>;
    typename SpinorIO<SP>::Hop sf, sb;
    uint32_t wf[F::kWords], wb[F::kWords];
    C<typename LinkReal<LP>::R> u[3][3];
    if constexpr (SP != P64 || PAIR64) {
        // all loads of both hops first: one memory round trip instead of two
        // (FP64 otherwise keeps the two trips: its registers would cut the occupancy)
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[MU], sf);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, p * 4 + MU, i, wf);
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[4 + MU], sb);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, (1 - p) * 4 + MU, nb[4 + MU], wb);
        more();
        __builtin_amdgcn_sched_barrier(0);   // keep the arithmetic below every load
        link_decode<LP, RECON>(wf, u);
        hop_fwd<MU>(sf, u, acc);
        link_decode<LP, RECON>(wb, u);
        hop_bwd<MU>(sb, u, acc);
    } else {
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[MU], sf);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, p * 4 + MU, i, wf);
        link_decode<LP, RECON>(wf, u);
        hop_fwd<MU>(sf, u, acc);
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[4 + MU], sb);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, (1 - p) * 4 + MU, nb[4 + MU], wb);
        more();
        link_decode<LP, RECON>(wb, u);
        hop_bwd<MU>(sb, u, acc);
    }
}

// Values computed here, not sunk to where they are used.
template <int N, typename R>
__device__ __forceinline__ void pin(C<R> (&x)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(x[k].r), "+v"(x[k].i));
}

// The one-lane kernels (k_wilson, the multi-RHS tile and the march along x0) add
// the hops of a site in one order: -0, +1, -1, +2, -2, +3, -3, +0.  The last is
// the one a march along x0 has last, so that all of them round alike.
// Two consecutive hops of that order: backward MUB, then forward MUF; the loads
// of both first, except for FP64, whose registers would cut the occupancy.
template <int SP, int LP, int RECON, int MUB, bool NT>
__device__ __forceinline__ void hop_chain(const WilsonArgs& a, int p, int32_t i, const int32_t nb[8],
                                          const SpinorView& vin, C<typename SpinorIO<SP>::R> acc[12]) {
    constexpr int MUF = (MUB + 1) & 3;
    using F = LinkFmt<LP, RECON>;
    typename SpinorIO<SP>::Hop sf, sb;
    uint32_t wf[F::kWords], wb[F::kWords];
    C<typename LinkReal<LP>::R> u[3][3];
    SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[4 + MUB], sb);
    link_load_words<LP, RECON, NT>(a.links, a.g.vh, (1 - p) * 4 + MUB, nb[4 + MUB], wb);
    if constexpr (SP != P64) {
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[MUF], sf);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, p * 4 + MUF, i, wf);
        __builtin_amdgcn_sched_barrier(0);   // keep the arithmetic below every load
    }
    link_decode<LP, RECON>(wb, u);
    hop_bwd<MUB>(sb, u, acc);
    if constexpr (SP == P64) {
        SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[MUF], sf);
        link_load_words<LP, RECON, NT>(a.links, a.g.vh, p * 4 + MUF, i, wf);
    }
    link_decode<LP, RECON>(wf, u);
    hop_fwd<MUF>(sf, u, acc);
}

__device__ __forceinline__ double coef(const Coef& c) { return c.d ? c.f * (*c.d) : c.f; }

// Tile order for cache reuse of the neighbour spinors.  In index order the
// tiles holding the x0 neighbours of a tile lie a whole x0 slice (S tiles)
// away, too far back for that slice's spinors to still be in L2.  With chunk c
// (c divides S) the position p of a launch is mapped to the tile
//   x0 = (p mod c N0) / c,  j = (p / c N0) c + p mod c,  tile = x0 S + j,
// i.e. c consecutive tiles of every x0 slice in turn: x0 neighbours are then c
// positions apart and x1 neighbours (s1 / tile sites apart) mostly inside the
// same chunk.  A permutation of the tiles: the arithmetic is unchanged.
__device__ __forceinline__ int32_t order_tile(int32_t p, const TileOrder& o) {
    if (o.c <= 0) return p;
    const int32_t k = (int32_t)fdiv((uint32_t)p, o.d_cn);
    const int32_t rem = p - k * o.cn;
    const int32_t x0 = (int32_t)fdiv((uint32_t)rem, o.d_c);
    return x0 * o.slice + k * o.c + (rem - x0 * o.c);
}

// Block index remap that gives each of the 8 XCDs (workgroups dispatched
// round-robin, linear id mod 8) one contiguous range of tiles, so that
// neighbour re-reads stay in that XCD's L2.
__device__ __forceinline__ unsigned xcd_remap(unsigned lin, unsigned total) {
    const unsigned x = lin & 7u;
    const unsigned q = total >> 3, r = total & 7u;
    const unsigned start = x * q + (x < r ? x : r);
    return start + (lin >> 3);
}

// Launch position -> (parity slot y, position within that parity).  With both
// parities in one launch (the full Q) the two parities of a tile take adjacent
// positions, so after the XCD remap they run on the same XCD at about the same
// time: the links one parity reads as forward links the other reads as backward
// links, and the second read finds them in that XCD's L2.  The position is then
// mapped to a tile by order_tile.
__device__ __forceinline__ int32_t parity_slot(unsigned lin, unsigned gx, unsigned gy, int& y) {
    if (gy == 2) {
        y = (int)(lin & 1u);
        return (int32_t)(lin >> 1);
    }
    y = 0;   // one output parity
    return (int32_t)lin;
}

template <int SP, int LP, int RECON, int BLOCK, bool NT>
__global__ void __launch_bounds__(BLOCK) k_wilson(WilsonArgs a) {
    using R = typename SpinorIO<SP>::R;
    __shared__ double red_lds[BLOCK / 64];
    unsigned lin = blockIdx.y * gridDim.x + blockIdx.x;
    if (a.xcd_remap) lin = xcd_remap(lin, gridDim.x * gridDim.y);
    int y;
    const int32_t pos = parity_slot(lin, gridDim.x, gridDim.y, y);
    const int32_t i = order_tile(pos, a.order) * BLOCK + threadIdx.x;
    const int p = a.p0 + y;
    double red = 0.0;
    if (i < a.g.vh) {
        const SiteCoord x = eo_coords(a.g, p, i);
        int32_t nb[8];
        eo_neighbours(a.g, i, x, nb);
        C<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        const SpinorView& vin = a.in[y];
        hop_chain<SP, LP, RECON, 0, NT>(a, p, i, nb, vin, acc);
        hop_chain<SP, LP, RECON, 1, NT>(a, p, i, nb, vin, acc);
        hop_chain<SP, LP, RECON, 2, NT>(a, p, i, nb, vin, acc);
        hop_chain<SP, LP, RECON, 3, NT>(a, p, i, nb, vin, acc);

        const R b = (R)a.b_hop;
        if (a.has_self) {
            C<R> sf[12];
            SpinorIO<SP>::load(a.self[y], (int64_t)a.self[y].site0 + i, sf);
            const R as = (R)a.a_self;
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = {as * sf[k].r + b * acc[k].r, as * sf[k].i + b * acc[k].i};
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = cscale(b, acc[k]);
        }
        if (a.gamma5) {
#pragma unroll
            for (int k = 6; k < 12; ++k) acc[k] = cneg(acc[k]);
        }
        const R c0 = (R)coef(a.c0);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = cscale(c0, acc[k]);
        for (int j = 0; j < a.nv; ++j) {
            C<R> vv[12];
            SpinorIO<SP>::load(a.v[j][y], (int64_t)a.v[j][y].site0 + i, vv);
            const R cj = (R)coef(a.cv[j]);
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = {acc[k].r + cj * vv[k].r, acc[k].i + cj * vv[k].i};
        }
        SpinorIO<SP>::store(a.out[y], (int64_t)a.out[y].site0 + i, acc);
        if (a.partials) {
            if constexpr (SP == P16) {
                // norm of what was stored (after F16 rounding)
                SpinorIO<SP>::load(a.out[y], (int64_t)a.out[y].site0 + i, acc);
            }
#pragma unroll
            for (int k = 0; k < 12; ++k) red += (double)acc[k].r * acc[k].r + (double)acc[k].i * acc[k].i;
        }
    }
    if (a.partials) {
        const double s = block_sum(red, red_lds);
        if (threadIdx.x == 0) a.partials[lin] = s;
    }
}

// Epilogue of the direction split: the part of the 64 outputs that wavefront w
// finishes, kN complex components from first(w).  F64: one spin component of
// each site; F32: the two 16-byte planes 2w, 2w+1 (wavefronts 0..2), so that
// every access is a full word; F16: plane w (wavefronts 0..2), whose stores wait
// for the site's scale, the largest of all 24 reals.
template <int SP> struct SplitPart;
template <> struct SplitPart<P64> {
    static constexpr int kN = 3;
    __device__ static __forceinline__ bool has(int) { return true; }
    __device__ static __forceinline__ void load(const SpinorView& v, int64_t s, int w, C<double> x[kN]) {
#pragma unroll
        for (int k = 0; k < kN; ++k) x[k] = SpinorIO<P64>::load_comp(v, s, kN * w + k);
    }
    __device__ static __forceinline__ void store(const SpinorView& v, int64_t s, int w, const C<double> x[kN]) {
#pragma unroll
        for (int k = 0; k < kN; ++k) SpinorIO<P64>::store_comp(v, s, kN * w + k, x[k]);
    }
};
template <> struct SplitPart<P32> {
    static constexpr int kN = 4;
    __device__ static __forceinline__ bool has(int w) { return w < 3; }
    __device__ static __forceinline__ void load(const SpinorView& v, int64_t s, int w, C<float> x[kN]) {
        SpinorIO<P32>::load_plane(v, s, 2 * w, x[0], x[1]);
        SpinorIO<P32>::load_plane(v, s, 2 * w + 1, x[2], x[3]);
    }
    __device__ static __forceinline__ void store(const SpinorView& v, int64_t s, int w, const C<float> x[kN]) {
        SpinorIO<P32>::store_plane(v, s, 2 * w, x[0], x[1]);
        SpinorIO<P32>::store_plane(v, s, 2 * w + 1, x[2], x[3]);
    }
};
template <> struct SplitPart<P16> {
    static constexpr int kN = 4;
    __device__ static __forceinline__ bool has(int w) { return w < 3; }
    __device__ static __forceinline__ void load(const SpinorView& v, int64_t s, int w, C<float> x[kN]) {
        SpinorIO<P16>::load_plane(v, s, w, x);
    }
};

// Direction-split variant for small lattices, where one lane per site leaves
// most SIMDs with a single wavefront: a workgroup of 4 wavefronts covers 64
// sites and wavefront w computes the two hops +-mu with mu = w (the direction is
// uniform per wavefront, so there is no divergence).  The four partial sums
// meet in LDS and are added in a fixed order; wavefront w then finishes its
// part of the 64 outputs (SplitPart).
//
// Bound by memory round trips, on small lattices entirely.  The same-site
// spinor and the up to NV = 3 extra vectors of the epilogue are therefore
// loaded together with the hops' spinors and links, not after the barrier one
// round trip each: one F32 sign apply on 24^3x48 14.2 -> 12.2 ms, the F32 Q
// there 75.0 -> 70.6 us, a mixed solve on 8^3x16 381-420 -> 332-360 ms (loads
// between the arithmetic and the barrier instead: 12.4 ms, 72.1 us and
// 349-389 ms, although that keeps 5 wavefronts per SIMD instead of 4).  NV = 0
// serves launches without extra vectors, whose registers the loads would cost.
// There FP64 fields with 8-real links load the same-site spinor after the barrier:
// 166 registers instead of 178 keep three wavefronts per SIMD through the links'
// decoding (24^3x48 Q 135.8 -> 122.5 us, dslash 71.7 -> 61.5, 32^3x64 dslash 223 -> 199).
// 12-real links stay at two either way, and 18-real ones lose more by the later load
// than a third wavefront gains (Q on 24^3x20 58.5 us, 63.8 with 140 registers).
// F16 shares the epilogue out by planes too and settles the site's scale with a
// second barrier: a whole spinor and three whole extra vectors in wavefront 0 took
// 160 registers in every wavefront, a plane of each takes 93 (5 wavefronts per SIMD
// instead of 3; one F16 sign apply on 24^3x48 9.34 -> 7.51 ms, on 16^3x32 1.97 -> 1.64
// ms, Q without extra vectors on 32^3x64 126 -> 121 us, the same bits).
template <int SP, int LP, int RECON, bool NT, int NV>
__global__ void __launch_bounds__(256) k_wilson_dirsplit(WilsonArgs a) {
    using R = typename SpinorIO<SP>::R;
    using Part = SplitPart<SP>;
    __shared__ C<R> part[4][12][64];
    __shared__ double red_lds[4];
    // every argument on the way to the first loads, read in one go: left to itself
    // the compiler reads them one by one where each is used, a dozen scalar
    // round trips in a row before the first spinor is asked for (mixed solve on
    // 8^3x16, one workgroup per CU, 333-349 -> 306-314 ms with this, the extra
    // vectors' views and the epilogue's scalars read ahead; FP64 Q on 24^3x48,
    // whose tile order now divides by multiplication too, 139.4 -> 134.6 us)
    WilsonArgs h;
    h.g = a.g;
    h.links = a.links;
    h.order = a.order;
    const unsigned gx = gridDim.x, gy = gridDim.y;
    const int p0 = a.p0, remap = a.xcd_remap, has_self = a.has_self;
    const char* in_base = a.in[0].base;
    const int32_t in_stride = a.in[0].stride, in0 = a.in[0].site0, in1 = a.in[1].site0;
    const char* self_base = a.self[0].base;
    const int32_t self0 = a.self[0].site0, self1 = a.self[1].site0;
    asm volatile("" ::"s"(h.g.n0), "s"(h.g.n1), "s"(h.g.n2), "s"(h.g.n3), "s"(h.g.nh3), "s"(h.g.s1), "s"(h.g.s0),
                 "s"(h.g.vh), "s"(h.g.d_nh3.m), "s"(h.g.d_nh3.s), "s"(h.g.d_n2.m), "s"(h.g.d_n2.s), "s"(h.g.d_n1.m),
                 "s"(h.g.d_n1.s), "s"(p0), "s"(remap), "s"(h.order.c), "s"(has_self), "s"(gx), "s"(gy), "s"(h.links), "s"(in_base),
                 "s"(in_stride), "s"(in0), "s"(in1), "s"(self_base), "s"(self0), "s"(self1));
    unsigned lin = blockIdx.y * gx + blockIdx.x;
    if (remap) lin = xcd_remap(lin, gx * gy);
    int y;
    const int32_t pos = parity_slot(lin, gx, gy, y);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t i = order_tile(pos, h.order) * 64 + lane;
    const int p = p0 + y;
    const bool active = i < h.g.vh;
    const SpinorView vin = {const_cast<char*>(in_base), in_stride, y ? in1 : in0, 0};
    const SpinorView vself = {const_cast<char*>(self_base), in_stride, y ? self1 : self0, 0};
    SpinorView vj[NV > 0 ? NV : 1];
    int nv = 0;
    if constexpr (NV > 0) {
        nv = a.nv;
        asm volatile("" : "+s"(nv));
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            vj[j] = a.v[j][0];
            int32_t s1 = a.v[j][1].site0;
            asm volatile("" : "+s"(vj[j].base), "+s"(vj[j].stride), "+s"(vj[j].site0), "+s"(s1));
            if (y) vj[j].site0 = s1;
        }
    }
    // the epilogue's scalars
    double as_d = a.a_self, b_d = a.b_hop, c0_f = a.c0.f;
    const double* c0_d = a.c0.d;
    int g5 = a.gamma5;
    SpinorView vout = a.out[0];
    int32_t out1 = a.out[1].site0;
    double* partials = a.partials;
    Coef cj[NV > 0 ? NV : 1];
#pragma unroll
    for (int j = 0; j < NV; ++j) cj[j] = a.cv[j];
    constexpr bool kSelfLate = SP == P64 && RECON == 8 && NV == 0;
    C<R> sf[Part::kN], vv[NV > 0 ? NV : 1][Part::kN];
    // the epilogue's operands, in flight with those of the hops
    auto epilogue_loads = [&]() {
        if (!kSelfLate && Part::has(w) && has_self) Part::load(vself, (int64_t)vself.site0 + i, w, sf);
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (Part::has(w) && j < nv) Part::load(vj[j], (int64_t)vj[j].site0 + i, w, vv[j]);
        // and its scalars: read behind the barrier, one by one, they cost a round trip each
        asm volatile("" : "+s"(as_d), "+s"(b_d), "+s"(c0_f), "+s"(c0_d), "+s"(g5), "+s"(vout.base), "+s"(vout.stride),
                     "+s"(vout.site0), "+s"(out1), "+s"(partials));
#pragma unroll
        for (int j = 0; j < NV; ++j) asm volatile("" : "+s"(cj[j].f), "+s"(cj[j].d));
    };
    if (active) {
        const SiteCoord x = eo_coords(h.g, p, i);
        int32_t nb[8];
        eo_neighbours(h.g, i, x, nb);
        C<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        switch (w) {
            case 0: hop_pair<SP, LP, RECON, 0, NT, RECON != 18>(h, p, i, nb, vin, acc, epilogue_loads); break;
            case 1: hop_pair<SP, LP, RECON, 1, NT, RECON != 18>(h, p, i, nb, vin, acc, epilogue_loads); break;
            case 2: hop_pair<SP, LP, RECON, 2, NT, RECON != 18>(h, p, i, nb, vin, acc, epilogue_loads); break;
            default: hop_pair<SP, LP, RECON, 3, NT, RECON != 18>(h, p, i, nb, vin, acc, epilogue_loads); break;
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) part[w][k][lane] = acc[k];
    }
    if (y) vout.site0 = out1;
    __syncthreads();
    double red = 0.0;
    const bool mine = active && Part::has(w);
    C<R> t[Part::kN];
    if (mine) {
        const R b = (R)b_d;
        const R as = (R)as_d;
        const R c0 = (R)coef(Coef{c0_f, c0_d});
        const int c1 = Part::kN * w;   // first component of this part
        if (kSelfLate && has_self) Part::load(vself, (int64_t)vself.site0 + i, w, sf);
#pragma unroll
        for (int k = 0; k < Part::kN; ++k) {
            const int c = c1 + k;
            t[k] = cadd(cadd(part[0][c][lane], part[1][c][lane]), cadd(part[2][c][lane], part[3][c][lane]));
            if (has_self) t[k] = {as * sf[k].r + b * t[k].r, as * sf[k].i + b * t[k].i};
            else t[k] = cscale(b, t[k]);
            if (g5 && c >= 6) t[k] = cneg(t[k]);
            t[k] = cscale(c0, t[k]);
        }
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if (j < nv) {
                const R cr = (R)coef(cj[j]);
#pragma unroll
                for (int k = 0; k < Part::kN; ++k) t[k] = {t[k].r + cr * vv[j][k].r, t[k].i + cr * vv[j][k].i};
            }
        }
    }
    float amax = 0.f;
    if constexpr (SP == P16) {
        __shared__ float amax_lds[3][64];
        if (mine) {
#pragma unroll
            for (int k = 0; k < Part::kN; ++k) amax = fmaxf(amax, fmaxf(fabsf(t[k].r), fabsf(t[k].i)));
            amax_lds[w][lane] = amax;
        }
        __syncthreads();
        amax = fmaxf(amax_lds[0][lane], fmaxf(amax_lds[1][lane], amax_lds[2][lane]));
    }
    if (mine) {
        const int64_t so = (int64_t)vout.site0 + i;
        if constexpr (SP == P16) SpinorIO<P16>::store_plane(vout, so, w, amax, t);   // leaves in t what was stored
        else Part::store(vout, so, w, t);
        if (partials) {
#pragma unroll
            for (int k = 0; k < Part::kN; ++k) red += (double)t[k].r * t[k].r + (double)t[k].i * t[k].i;
        }
    }
    if (partials) {
        const double s = block_sum(red, red_lds);
        if (threadIdx.x == 0) partials[lin] = s;
    }
}

// Links of a multi-right-hand-side tile in LDS, per direction a block of
// planes of 64 sites (lane l touches consecutive words).  F32/F16 links and the
// 8-real FP64 ones are decoded to 18 reals once per tile (the reconstructions
// then run once per link, not once per right-hand side).  For 8 FP64 reals, sine,
// cosine, square roots and a division per link, that is most of the work, and in
// the field loop it spilled (480 bytes a lane, one wavefront per SIMD): 12 fields
// on 24^3x48 4432 -> 1175 us, 8 on 16^3x32 474 -> 151 us, the same bits, with 72
// KiB of LDS and the two wavefronts per SIMD that the registers allow.  12- and
// 18-real FP64 links stay in their stored words and are decoded per right-hand
// side: a 12-real tile needs 48 KiB, and its cross products cost less than reading
// the third row back (12 fields 1153 us against 1178, 60 fields 5.70 against 5.82 ms).
template <int LP, int RECON>
struct StagedLinks {
    using LR = typename LinkReal<LP>::R;
    static constexpr bool kDecoded = LP != P64 || RECON == 8;
    static constexpr int kWords = kDecoded ? 18 * (int)(sizeof(LR) / 4) : LinkFmt<LP, RECON>::kWords;
    __device__ static __forceinline__ void put(uint32_t* lw, int dir, int lane, const uint32_t words[]) {
        if constexpr (kDecoded) {
            C<LR> u[3][3];
            link_decode<LP, RECON>(words, u);
            LR* d = reinterpret_cast<LR*>(lw) + dir * 18 * 64 + lane;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    d[(2 * (3 * r + c)) * 64] = u[r][c].r;
                    d[(2 * (3 * r + c) + 1) * 64] = u[r][c].i;
                }
        } else {
#pragma unroll
            for (int k = 0; k < kWords; ++k) lw[(dir * kWords + k) * 64 + lane] = words[k];
        }
    }
    __device__ static __forceinline__ void get(const uint32_t* lw, int dir, int lane, C<LR> u[3][3]) {
        if constexpr (kDecoded) {
            const LR* d = reinterpret_cast<const LR*>(lw) + dir * 18 * 64 + lane;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) u[r][c] = {d[(2 * (3 * r + c)) * 64], d[(2 * (3 * r + c) + 1) * 64]};
        } else {
            uint32_t words[kWords];
#pragma unroll
            for (int k = 0; k < kWords; ++k) words[k] = lw[(dir * kWords + k) * 64 + lane];
            link_decode<LP, RECON>(words, u);
        }
    }
};

// Many right-hand sides on one gauge field: a workgroup of 4 wavefronts owns
// 64 output sites; it first stages the 8 links of each site into LDS (forward
// links at the tile's own sites, backward links at the neighbours; see
// StagedLinks), then wavefront q computes right-hand sides q, q+4, q+8, ... for
// the 64 sites, reading the links from LDS.  Links leave HBM once per apply
// instead of once per right-hand side; every spinor load of a
// wavefront is one right-hand side's 64 consecutive sites.  The per-site
// arithmetic is that of k_wilson (same hop order and epilogue), so results
// match the one-lane-per-site kernel bit for bit.
//
// One tile: output parity p, sites 64*tile .. 64*tile+63 of that parity, and
// right-hand sides r0 .. r1-1.  The views address right-hand side 0;
// right-hand side r sits r * rhs_bytes further.  has_self = false: no
// same-site term.  Must be reached by all 256 threads of the workgroup (it
// synchronises once).  PIN: the sums of each two hops are formed before the next
// two (see k_wilson_multi).
template <int SP, int LP, int RECON, bool NT, bool PIN = false>
__device__ __forceinline__ void mrhs_tile(const GeomK& g, const char* links, int p, int32_t tile,
                                          const SpinorView& in, const SpinorView& self, bool has_self,
                                          const SpinorView& out, double a_self, double b_hop, int gamma5, double c0d,
                                          int r0, int r1, uint32_t* lw, int nv = 0, const SpinorView* v = nullptr,
                                          int vstride = 1, const Coef* cv = nullptr) {
    using R = typename SpinorIO<SP>::R;
    using LR = typename LinkReal<LP>::R;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int32_t i = tile * 64 + lane;
    const bool active = i < g.vh;
    int32_t nb[8];
    using SL = StagedLinks<LP, RECON>;
    if (active) {
        const SiteCoord x = eo_coords(g, p, i);
        eo_neighbours(g, i, x, nb);
        // wavefront w stages the forward link mu = w and the backward link mu = w
        uint32_t words[LinkFmt<LP, RECON>::kWords];
        link_load_words<LP, RECON, NT>(links, g.vh, p * 4 + w, i, words);
        SL::put(lw, w, lane, words);
        link_load_words<LP, RECON, NT>(links, g.vh, (1 - p) * 4 + w, nb[4 + w], words);
        SL::put(lw, 4 + w, lane, words);
    }
    __syncthreads();
    if (!active) return;
#pragma unroll 1
    for (int r = r0 + w; r < r1; r += 4) {
        // re-read links from LDS for every right-hand side instead of letting
        // them be hoisted into registers (which would cost occupancy)
        int lo = lane;
        asm volatile("" : "+v"(lo));
        SpinorView vin = in;
        vin.base += (int64_t)r * vin.rhs_bytes;
        C<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        // the order of hop_chain, the spinor loads of two hops first (one memory
        // round trip per pair; FP64: one per hop, for its registers)
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const int mf = (mu + 1) & 3;
            typename SpinorIO<SP>::Hop sf, sb;
            C<LR> u[3][3];
            SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[4 + mu], sb);
            if constexpr (SP != P64) {
                SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[mf], sf);
                __builtin_amdgcn_sched_barrier(0);
            }
            SL::get(lw, 4 + mu, lo, u);
            if (mu == 0) hop_bwd<0>(sb, u, acc);
            if (mu == 1) hop_bwd<1>(sb, u, acc);
            if (mu == 2) hop_bwd<2>(sb, u, acc);
            if (mu == 3) hop_bwd<3>(sb, u, acc);
            if constexpr (SP == P64) SpinorIO<SP>::load_hop(vin, (int64_t)vin.site0 + nb[mf], sf);
            SL::get(lw, mf, lo, u);
            if (mf == 0) hop_fwd<0>(sf, u, acc);
            if (mf == 1) hop_fwd<1>(sf, u, acc);
            if (mf == 2) hop_fwd<2>(sf, u, acc);
            if (mf == 3) hop_fwd<3>(sf, u, acc);
            if constexpr (PIN) pin(acc);
        }
        const R b = (R)b_hop;
        if (has_self) {
            SpinorView vs = self;
            vs.base += (int64_t)r * vs.rhs_bytes;
            C<R> sf[12];
            SpinorIO<SP>::load(vs, (int64_t)vs.site0 + i, sf);
            const R as = (R)a_self;
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = {as * sf[k].r + b * acc[k].r, as * sf[k].i + b * acc[k].i};
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = cscale(b, acc[k]);
        }
        if (gamma5) {
#pragma unroll
            for (int k = 6; k < 12; ++k) acc[k] = cneg(acc[k]);
        }
        const R c0 = (R)c0d;
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = cscale(c0, acc[k]);
        for (int j = 0; j < nv; ++j) {
            SpinorView vj = v[j * vstride];
            vj.base += (int64_t)r * vj.rhs_bytes;
            C<R> vv[12];
            SpinorIO<SP>::load(vj, (int64_t)vj.site0 + i, vv);
            const R cj = (R)coef(cv[j]);
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = {acc[k].r + cj * vv[k].r, acc[k].i + cj * vv[k].i};
        }
        SpinorView vo = out;
        vo.base += (int64_t)r * vo.rhs_bytes;
        SpinorIO<SP>::store(vo, (int64_t)vo.site0 + i, acc);
    }
}

// Work order of the multi-right-hand-side launch: a 1-D grid of tiles x ny
// output parities x ngroups groups of `rg` right-hand sides.  Group-major
// order runs every tile for one group before the next group (the spinors
// re-read by neighbouring tiles are then those of rg fields only, so they stay
// in L2; links are read once per group); tile-major order runs the groups of a
// tile next to each other (they share the tile's links in L2).
// XCD-group order (group_major = 2, ngroups dividing 8): workgroup b runs on
// XCD b mod 8 (the dispatcher's round robin); XCD x takes group x mod ngroups
// and part x / ngroups of the tile list, in order.  The XCDs holding the same
// part walk the same tiles at about the same time, so each tile's links come
// from HBM once and from the shared last-level cache for the other groups,
// while each XCD's L2 holds the neighbour spinors of its own rg fields only.
struct MrhsGrid {
    int32_t tiles;       // tiles of 64 sites per parity
    int ny;              // output parities (1 or 2)
    int rg;              // right-hand sides per workgroup
    int ngroups;
    int group_major;     // 0 tile-major, 1 group-major, 2 XCD groups
    int nrhs;
    int32_t per_part;    // XCD groups: tile positions per part
};

template <int SP, int LP, int RECON, bool NT>
__global__ void __launch_bounds__(256) k_wilson_mrhs(WilsonArgs a, MrhsGrid m) {
    extern __shared__ uint32_t lw[];   // [8 dirs][StagedLinks words][64 sites]
    // the arguments on the way to the first loads in one go (see k_wilson_dirsplit;
    // 12 F16 fields on 24^3x48 351 -> 332 us, 4 instead of 3 wavefronts per SIMD
    // as the views are no longer re-read from memory in the field loop)
    const GeomK g = a.g;
    const char* links = a.links;
    SpinorView vin = a.in[0], vself = a.self[0], vout = a.out[0];
    const int32_t in1 = a.in[1].site0, self1 = a.self[1].site0, out1 = a.out[1].site0;
    const TileOrder order = a.order;
    const unsigned gx = gridDim.x;
    asm volatile("" ::"s"(g.n0), "s"(g.n1), "s"(g.n2), "s"(g.n3), "s"(g.nh3), "s"(g.s1), "s"(g.s0), "s"(g.vh),
                 "s"(g.d_nh3.m), "s"(g.d_nh3.s), "s"(g.d_n2.m), "s"(g.d_n2.s), "s"(g.d_n1.m), "s"(g.d_n1.s), "s"(links),
                 "s"(a.p0), "s"(a.xcd_remap), "s"(order.c), "s"(order.cn), "s"(order.slice), "s"(order.d_c.m),
                 "s"(order.d_c.s), "s"(order.d_cn.m), "s"(order.d_cn.s), "s"(gx));
    asm volatile("" ::"s"(m.tiles), "s"(m.ny), "s"(m.rg), "s"(m.ngroups), "s"(m.group_major), "s"(m.nrhs),
                 "s"(vin.base), "s"(vin.stride), "s"(vin.site0), "s"(in1), "s"(vin.rhs_bytes), "s"(a.has_self));
    const unsigned per_group = (unsigned)(m.ny * m.tiles);
    unsigned grp, rem;
    if (m.group_major == 2) {
        const unsigned x = blockIdx.x & 7u, k = blockIdx.x >> 3;
        grp = x % (unsigned)m.ngroups;
        rem = (x / (unsigned)m.ngroups) * (unsigned)m.per_part + k;
        if (rem >= per_group) return;   // the whole workgroup: before any barrier
    } else {
        unsigned lin = blockIdx.x;
        if (a.xcd_remap) lin = xcd_remap(lin, gx);
        if (m.group_major) {
            grp = lin / per_group;
            rem = lin - grp * per_group;
        } else {
            rem = lin / (unsigned)m.ngroups;
            grp = lin - rem * (unsigned)m.ngroups;
        }
    }
    int y = 0;
    int32_t pos = (int32_t)rem;
    if (m.ny == 2) {
        y = (int)(rem & 1u);
        pos = (int32_t)(rem >> 1);
    }
    const int32_t tile = order_tile(pos, order);
    const int r0 = (int)grp * m.rg;
    const int r1 = min(m.nrhs, r0 + m.rg);
    if (y) {
        vin.site0 = in1;
        vself.site0 = self1;
        vout.site0 = out1;
    }
    mrhs_tile<SP, LP, RECON, NT>(g, links, a.p0 + y, tile, vin, vself, a.has_self != 0, vout, a.a_self,
                                 a.b_hop, a.gamma5, coef(a.c0), r0, r1, lw, a.nv, &a.v[0][y], 2, a.cv);
}

template <int SP, int LP, int RECON>
size_t mrhs_lds_bytes() {
    return (size_t)8 * StagedLinks<LP, RECON>::kWords * 64 * sizeof(uint32_t);
}

// FP64 18-real links need 72 KiB of LDS per workgroup (of the 160 KiB per CU):
// opt in above the default 64 KiB limit.
template <typename K>
hipError_t allow_lds(K kernel, size_t lds) {
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds);
}

template <int SP, int LP, int RECON, bool NT>
hipError_t launch_mrhs_nt(const WilsonArgs& a, const MrhsGrid& m, hipStream_t st) {
    const dim3 grid(m.group_major == 2 ? (unsigned)(8 * (int64_t)m.per_part)
                                       : (unsigned)((int64_t)m.tiles * m.ny * m.ngroups));
    const size_t lds = mrhs_lds_bytes<SP, LP, RECON>();
    const hipError_t e = allow_lds(&k_wilson_mrhs<SP, LP, RECON, NT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_wilson_mrhs<SP, LP, RECON, NT>), grid, dim3(256), lds, st, a, m);
    return hipGetLastError();
}

// non-temporal link loads (automatic: when every link is read once, i.e. one
// output parity (ny = 1) and one group of right-hand sides)
template <int SP, int LP, int RECON>
hipError_t launch_mrhs_fmt(const WilsonArgs& a, const MrhsGrid& m, int link_nt, hipStream_t st) {
    const bool nt = link_nt < 0 ? (m.ny == 1 && m.ngroups == 1) : link_nt != 0;
    return nt ? launch_mrhs_nt<SP, LP, RECON, true>(a, m, st) : launch_mrhs_nt<SP, LP, RECON, false>(a, m, st);
}

// Many F32 right-hand sides on one gauge field, full Q, as a march along x0.
//
// The multi-RHS stencil is bound by what misses the L2s (about 6 TB/s on this
// card, from the last-level cache as from HBM).  In the tile form above a
// spinor misses 3 to 4 times: its x0 neighbours lie a whole slice of tiles
// away, and 4 MB of L2 per XCD do not hold what 128 workgroups of several
// fields read between the uses.  Here a workgroup of 4 wavefronts (one field
// each) owns a column of 64 sites of one parity per slice and walks T slices:
//   * psi(t - 1) and psi(t) of the column stay in registers, so a site takes 7
//     spinor loads instead of 9, and its x0 link one load instead of two;
//   * out(t - 1) gets its last hop (+0, which reads psi(t)) in step t, so that
//     every load of slice t, from the column itself and from the columns next to
//     it, falls into the same step and all but the first find it in L2.
// The 7 links of a step (fields share them) go to LDS, two buffers in turn, one
// barrier per step.  The hops, their order and the epilogue are those of
// k_wilson, so the results equal it bit for bit.  Outputs are stored with the
// non-temporal hint: nothing in the launch reads them.  About 235 registers, two
// wavefronts per SIMD.
// Measured, tile form in its default order and in its fastest one -> march, 12 fields:
// 24^3x48, 12-real links, 640 and 570 -> 521 us; 32^3x64, 12-real links, 2000 in the
// fastest -> 1759, 18-real links 2180 (6 fields per workgroup, 10.1 GB of L2 misses) and
// 2090 (12 fields, 13.5 GB) -> 1917 us (10.8 GB).  Launches that fuse
// three vectors gain nothing from it: on 24^3x48 1026 us, 1028 in the default tile order,
// 907 in the fastest.  Tried and not kept: the next slice's x1 neighbours in flight
// across the barrier (spills); FP64 (its registers); F16 fields (375 us against 332 us:
// half the traffic, and the tile form's four wavefronts per SIMD hide more).
struct MarchArgs {
    GeomK g;
    const char* links;
    const char* in;            // full fields, right-hand side 0
    char* out;
    const char* v[3];
    int64_t rhs_bytes;         // of every field
    int64_t plane;             // bytes between planes
    double a_self;
    Coef c0;
    Coef cv[3];
    int nrhs, ngroups;
    int32_t tiles;             // tiles of 64 sites per parity and x0 slice
    int32_t T, nseg;           // slices per segment, segments
};

template <int LP, int RECON, int NV>
__global__ void __launch_bounds__(256, 2) k_wilson_march(MarchArgs a) {
    using R = float;
    using IO = SpinorIO<P32>;
    using Hop = typename IO::Hop;
    using LR = typename LinkReal<LP>::R;
    using F = LinkFmt<LP, RECON>;
    using SL = StagedLinks<LP, RECON>;
    constexpr int kBuf = 7 * SL::kWords * 64;
    extern __shared__ uint32_t lw[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned lin = xcd_remap(blockIdx.x, gridDim.x);
    const int par = (int)(lin & 1u);
    lin >>= 1;
    const int32_t tile = (int32_t)(lin % (unsigned)a.tiles);
    lin /= (unsigned)a.tiles;
    const int seg = (int)(lin % (unsigned)a.nseg);
    const int grp = (int)(lin / (unsigned)a.nseg);
    // the fields split evenly over the groups, at most 4 each; a wavefront
    // without one still stages links
    const int r0 = grp * a.nrhs / a.ngroups, r1 = (grp + 1) * a.nrhs / a.ngroups;
    const int r = r0 + w;
    const bool field = r < r1;
    const GeomK& g = a.g;
    const int32_t jt = tile * 64 + lane;
    const bool active = jt < g.s0;
    const int32_t j = min(jt, g.s0 - 1);
    // offsets of the in-slice neighbours: constant along x0
    int32_t d[8];
    {
        const uint32_t q = fdiv((uint32_t)j, g.d_nh3);
        const int32_t x3h = j - (int32_t)q * g.nh3;
        const uint32_t x1 = fdiv(q, g.d_n2);
        const int32_t x2 = (int32_t)q - (int32_t)x1 * g.n2;
        const int bit = (par + (int)x1 + x2) & 1;
        d[1] = ((int32_t)x1 == g.n1 - 1) ? -(g.n1 - 1) * g.s1 : g.s1;
        d[5] = (x1 == 0) ? (g.n1 - 1) * g.s1 : -g.s1;
        d[2] = (x2 == g.n2 - 1) ? -(g.n2 - 1) * g.nh3 : g.nh3;
        d[6] = (x2 == 0) ? (g.n2 - 1) * g.nh3 : -g.nh3;
        d[3] = bit == 0 ? 0 : (x3h == g.nh3 - 1) ? 1 - g.nh3 : 1;
        d[7] = bit == 1 ? 0 : (x3h == 0) ? g.nh3 - 1 : -1;
    }
    const int32_t dbw = w == 1 ? d[5] : w == 2 ? d[6] : d[7];
    const R as = (R)a.a_self, b = R(-0.5), c0 = (R)coef(a.c0);
    R cv[NV > 0 ? NV : 1];
#pragma unroll
    for (int k = 0; k < NV; ++k) cv[k] = (R)coef(a.cv[k]);
    const int t0 = seg * a.T;
    const int t1 = min(g.n0, t0 + a.T);
    int p = (par + t0) & 1;
    const char* in = a.in + (int64_t)(field ? r : r0) * a.rhs_bytes;
    uint32_t wf[F::kWords], wb[F::kWords];
    // links of step t (sites of parity pp in slice t): wavefront 0 the x0 links of
    // slice t - 1, wavefront k the links k of the sites and of their neighbours x - k
    auto link_loads = [&](int pp, int t) {
        const int32_t tt = min(t, t1 - 1);
        const int32_t i = tt * g.s0 + j;
        const int32_t im = (t == 0 ? g.n0 - 1 : t - 1) * g.s0 + j;
        link_load_words<LP, RECON>(a.links, g.vh, w == 0 ? (1 - pp) * 4 : pp * 4 + w, w == 0 ? im : i, wf);
        if (w > 0) link_load_words<LP, RECON>(a.links, g.vh, (1 - pp) * 4 + w, i + dbw, wb);
    };
    auto link_stage = [&](uint32_t* buf) {
        SL::put(buf, w, lane, wf);
        if (w > 0) SL::put(buf, 3 + w, lane, wb);
    };
    auto own = [&](int pp, int t) { return 16u * (uint32_t)(pp * g.vh + t * g.s0 + j); };
    link_loads(p, t0);
    Hop cur, prev;
    C<R> q[12];   // out(t - 1) but for its last hop, then out(t)
    IO::load_hop_at(in, a.plane, own(1 - p, t0 == 0 ? g.n0 - 1 : t0 - 1), prev);
    IO::load_hop_at(in, a.plane, own(p, t0), cur);
#pragma unroll
    for (int k = 0; k < 12; ++k) q[k] = {R(0), R(0)};
    link_stage(lw);
    int cb = 0;
#pragma unroll 1
    for (int t = t0; t <= t1; ++t) {
        __syncthreads();
        const uint32_t* buf = lw + cb * kBuf;
        const uint32_t ob = own(1 - p, t);
        Hop s1, s2, s3, s4, nx;
        C<LR> u[3][3];
        C<R> acc[12];
        if (t < t1) link_loads(1 - p, t + 1);
        if (field) {
            Hop vv[NV > 0 ? NV : 1];
            if (NV > 0) {
                // slice t0 has nothing to finish yet: it loads its own sites' words
                const uint32_t om = t > t0 ? own(1 - p, t - 1) : own(p, t);
#pragma unroll
                for (int k = 0; k < NV; ++k)
                    IO::load_hop_at(a.v[k] + (int64_t)r * a.rhs_bytes, a.plane, om, vv[k]);
            }
            if (NV == 0 && t < t1) {
                IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[1], s1);
                IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[5], s2);
            }
            __builtin_amdgcn_sched_barrier(0);
            SL::get(buf, 0, lane, u);
            hop_fwd<0>(cur, u, q);
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
            hop_bwd<0>(prev, u, acc);
            pin(acc);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const C<R> x = prev.get(k);
                q[k] = {as * x.r + b * q[k].r, as * x.i + b * q[k].i};
                if (k >= 6) q[k] = cneg(q[k]);
                q[k] = cscale(c0, q[k]);
            }
            pin(q);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NV > 0) {
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int c = 0; c < 12; ++c) {
                        const C<R> x = vv[k].get(c);
                        q[c] = {q[c].r + cv[k] * x.r, q[c].i + cv[k] * x.i};
                    }
                pin(q);
            }
            if (active && t > t0) IO::store_nt(a.out + (int64_t)r * a.rhs_bytes, a.plane, own(1 - p, t - 1), q);
        }
        if (t == t1) break;
        if (field) {
            if (NV > 0) {
                IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[1], s1);
                IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[5], s2);
            }
            IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[2], s3);
            IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[6], s4);
            __builtin_amdgcn_sched_barrier(0);
            SL::get(buf, 1, lane, u);
            hop_fwd<1>(s1, u, acc);
            SL::get(buf, 4, lane, u);
            hop_bwd<1>(s2, u, acc);
            pin(acc);
            IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[3], s1);
            IO::load_hop_at(in, a.plane, ob + 16u * (uint32_t)d[7], s2);
            __builtin_amdgcn_sched_barrier(0);
            SL::get(buf, 2, lane, u);
            hop_fwd<2>(s3, u, acc);
            SL::get(buf, 5, lane, u);
            hop_bwd<2>(s4, u, acc);
            pin(acc);
            IO::load_hop_at(in, a.plane, own(1 - p, t + 1 == g.n0 ? 0 : t + 1), nx);
            __builtin_amdgcn_sched_barrier(0);
            SL::get(buf, 3, lane, u);
            hop_fwd<3>(s1, u, acc);
            SL::get(buf, 6, lane, u);
            hop_bwd<3>(s2, u, acc);
            pin(acc);
            prev = cur;
            cur = nx;
#pragma unroll
            for (int k = 0; k < 12; ++k) q[k] = acc[k];
        }
        cb ^= 1;   // the other buffer was last read before this step's barrier
        link_stage(lw + cb * kBuf);
        p = 1 - p;
    }
}

template <int LP, int RECON>
hipError_t launch_march(const WilsonArgs& a, int nrhs, hipStream_t st) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    MarchArgs m;
    memset(&m, 0, sizeof(m));
    m.g = a.g;
    m.links = a.links;
    m.in = a.in[0].base;
    m.out = a.out[0].base;
    m.rhs_bytes = a.in[0].rhs_bytes;
    m.plane = (int64_t)a.in[0].stride * 16;
    for (int k = 0; k < a.nv; ++k) {
        m.v[k] = a.v[k][0].base;
        m.cv[k] = a.cv[k];
    }
    m.a_self = a.a_self;
    m.c0 = a.c0;
    m.nrhs = nrhs;
    m.ngroups = (nrhs + 3) / 4;
    m.tiles = (a.g.s0 + 63) / 64;
    m.T = march_slices(a.g.n0, 2 * (int64_t)m.tiles * m.ngroups, 2 * cus);
    m.nseg = (a.g.n0 + m.T - 1) / m.T;
    const dim3 grid(2u * (unsigned)m.tiles * (unsigned)m.nseg * (unsigned)m.ngroups);
    const size_t lds = (size_t)2 * 7 * StagedLinks<LP, RECON>::kWords * 64 * sizeof(uint32_t);
    auto go = [&](auto kernel) -> hipError_t {
        const hipError_t er = allow_lds(kernel, lds);
        if (er != hipSuccess) return er;
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, m);
        return hipGetLastError();
    };
    switch (a.nv) {
        case 0: return go(&k_wilson_march<LP, RECON, 0>);
        case 2: return go(&k_wilson_march<LP, RECON, 2>);
        default: return go(&k_wilson_march<LP, RECON, 3>);
    }
}

// Q on several lattices (each with its own links and right-hand sides) in one
// persistent launch: the tiles of all lattices (both output parities) form one
// list; a grid of a fixed number of workgroups (a small multiple of what the
// device holds at once, independent of the lattices) walks it, workgroup b
// taking one contiguous chunk of tiles (chunks adjacent in the list go to
// workgroups on the same XCD), and each tile runs mrhs_tile with the epilogue
// of Q.
//
// Bound like the tiles by L2 misses and their latency.  With the epilogue's constants
// known the compiler keeps the products of all eight hops of an F16 field in registers
// and scales them at the end: 220 registers, two wavefronts per SIMD, 1 field on
// 32^3x64 337 us.  Formed after every two hops (PIN), 117 registers and four: 222 us
// (2 fields on 24^3x48 131 -> 88 us, 4 fields 170 -> 144; 12 fields on lattices below
// 10^4 sites 12.7 -> 13.5).  The one-lane kernels and k_wilson_mrhs, at 104 to 164
// registers, lose 1 to 3% by it.
template <int SP, int LP, int RECON>
__global__ void __launch_bounds__(256) k_wilson_multi(MultiArgs a) {
    extern __shared__ uint32_t lw[];
    const unsigned lin = xcd_remap(blockIdx.x, gridDim.x);
    const int chunk = (a.total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int t0 = (int)lin * chunk;
    const int t1 = min(a.total, t0 + chunk);
    for (int t = t0; t < t1; ++t) {
        int j = 0;
        while (j + 1 < a.njobs && t >= a.job[j + 1].tile0) ++j;
        const QJob& J = a.job[j];
        const int local = t - J.tile0;
        const int y = local / J.tiles;
        const int32_t tile = local - y * J.tiles;
        mrhs_tile<SP, LP, RECON, false, SP == P16>(J.g, J.links, y, tile, J.in[y], J.self[y], true, J.out[y], J.a_self,
                                                   -0.5, 1, 1.0, 0, J.nrhs, lw);
        __syncthreads();   // the next tile overwrites the staged links
    }
}

std::atomic<int> g_multi_grid{4};

template <int SP, int LP, int RECON>
hipError_t launch_multi_fmt(const MultiArgs& a, hipStream_t st) {
    const size_t lds = mrhs_lds_bytes<SP, LP, RECON>();
    auto kernel = &k_wilson_multi<SP, LP, RECON>;
    hipError_t e = allow_lds(kernel, lds);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 0, per_cu = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel), 256, lds)) !=
        hipSuccess)
        return e;
    // a multiple (default 4) of the workgroups the device holds at once: one
    // resident set walking long chunks leaves each workgroup a serial chain of
    // memory round trips; a larger grid overlaps them and still bounds the grid
    const int grid = std::max(1, std::min(a.total, multi_grid_factor() * std::max(1, per_cu) * cus));
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), lds, st, a);
    return hipGetLastError();
}

template <int SP, int LP, int RECON, bool NT>
hipError_t launch_nt(const WilsonArgs& a, int ny, int block, hipStream_t st) {
    if (block == 0) {
        // direction split: 64 sites per workgroup of 4 wavefronts
        const dim3 grid((unsigned)((a.g.vh + 63) / 64), ny);
        if constexpr (!NT) {
            if (a.nv > 0) {
                hipLaunchKernelGGL((k_wilson_dirsplit<SP, LP, RECON, NT, 3>), grid, dim3(256), 0, st, a);
                return hipGetLastError();
            }
        } else if (a.nv > 0) {
            return launch_nt<SP, LP, RECON, false>(a, ny, block, st);   // extra vectors: one instance per format
        }
        hipLaunchKernelGGL((k_wilson_dirsplit<SP, LP, RECON, NT, 0>), grid, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    const unsigned nbx = (unsigned)((a.g.vh + block - 1) / block);
    const dim3 grid(nbx, ny);
    switch (block) {
        case 64: hipLaunchKernelGGL((k_wilson<SP, LP, RECON, 64, NT>), grid, dim3(64), 0, st, a); break;
        case 128: hipLaunchKernelGGL((k_wilson<SP, LP, RECON, 128, NT>), grid, dim3(128), 0, st, a); break;
        default: hipLaunchKernelGGL((k_wilson<SP, LP, RECON, 256, NT>), grid, dim3(256), 0, st, a); break;
    }
    return hipGetLastError();
}

// one output parity (ny = 1) reads every link once: non-temporal link loads
template <int SP, int LP, int RECON>
hipError_t launch_fmt(const WilsonArgs& a, int ny, int block, hipStream_t st) {
    return ny == 1 ? launch_nt<SP, LP, RECON, true>(a, ny, block, st)
                   : launch_nt<SP, LP, RECON, false>(a, ny, block, st);
}

}  // namespace

namespace ndq {

int wilson_blocks(const ndq_geom* g, int block, int ny) {
    const int per = block == 0 ? 64 : block;
    return ((g->vh + per - 1) / per) * ny;
}

hipError_t launch_wilson(int sprec, int lprec, int recon, const WilsonArgs& args, int ny, int block,
                         hipStream_t st) {
    WilsonArgs a = args;
    int order = default_order(a.g, sprec, ny);
    if (block < 0) {
        const Tuning t = launch_tuning(a.g, sprec, lprec, recon, ny);
        block = t.block;
        a.xcd_remap = t.xcd_remap;
        order = t.order;
    }
    if (order) {
        const int lanes = block == 0 ? 64 : block;
        a.order = make_order((a.g.vh + lanes - 1) / lanes, a.g.n0, tile_order(a.g, lanes));
    }
    const int key = sprec * 1000 + lprec * 100 + recon;
    switch (key) {
        case P64 * 1000 + P64 * 100 + 18: return launch_fmt<P64, P64, 18>(a, ny, block, st);
        case P64 * 1000 + P64 * 100 + 12: return launch_fmt<P64, P64, 12>(a, ny, block, st);
        case P64 * 1000 + P64 * 100 + 8: return launch_fmt<P64, P64, 8>(a, ny, block, st);
        case P32 * 1000 + P32 * 100 + 18: return launch_fmt<P32, P32, 18>(a, ny, block, st);
        case P32 * 1000 + P32 * 100 + 12: return launch_fmt<P32, P32, 12>(a, ny, block, st);
        case P32 * 1000 + P32 * 100 + 8: return launch_fmt<P32, P32, 8>(a, ny, block, st);
        case P32 * 1000 + P16 * 100 + 18: return launch_fmt<P32, P16, 18>(a, ny, block, st);
        case P32 * 1000 + P16 * 100 + 12: return launch_fmt<P32, P16, 12>(a, ny, block, st);
        case P16 * 1000 + P32 * 100 + 18: return launch_fmt<P16, P32, 18>(a, ny, block, st);
        case P16 * 1000 + P32 * 100 + 12: return launch_fmt<P16, P32, 12>(a, ny, block, st);
        case P16 * 1000 + P32 * 100 + 8: return launch_fmt<P16, P32, 8>(a, ny, block, st);
        case P16 * 1000 + P16 * 100 + 18: return launch_fmt<P16, P16, 18>(a, ny, block, st);
        case P16 * 1000 + P16 * 100 + 12: return launch_fmt<P16, P16, 12>(a, ny, block, st);
        default: return hipErrorInvalidValue;
    }
}

namespace {
// Launches the march can take: full F32 fields, Q with the same field as stencil
// input and same-site term, 0, 2 or 3 extra vectors, 32-bit byte offsets.
// Extra vectors from 8 fields on: the march reads them after the barrier of a step,
// the tile form has more wavefronts to hide that.  D_N on 24^3x48, every second launch
// with 2 or 3 vectors, marching in all launches against the tile form in all: 3
// fields 1.00 of its time, 6 1.03, 7 1.11, 8 0.92, 9 0.79, 12 0.93, although the
// launches without vectors take 0.87 to 0.97.  (In the tiles' default order; the fastest
// one, chunk -1, makes 12 fields on 24^3x48 573 + 907 us as tiles, 540 + 1026 marching.)
bool march_fits(const WilsonArgs& a, int sprec, int ny, int nrhs) {
    if (sprec != P32 || ny != 2 || a.p0 != 0 || !a.has_self || !a.gamma5 || a.b_hop != -0.5 || a.partials ||
        a.nv == 1 || nrhs < (a.nv > 0 ? 8 : 3) || (int64_t)a.g.vh * 32 >= INT32_MAX)
        return false;
    const int32_t stride = 2 * a.g.vh;
    for (int p = 0; p < 2; ++p) {
        const SpinorView *in = &a.in[p], *self = &a.self[p], *out = &a.out[p];
        if (in->base != a.in[0].base || self->base != a.in[0].base || out->base != a.out[0].base ||
            in->site0 != (1 - p) * a.g.vh || self->site0 != p * a.g.vh || out->site0 != p * a.g.vh ||
            in->stride != stride || out->stride != stride || out->rhs_bytes != a.in[0].rhs_bytes)
            return false;
        for (int k = 0; k < a.nv; ++k)
            if (a.v[k][p].base != a.v[k][0].base || a.v[k][p].site0 != p * a.g.vh || a.v[k][p].stride != stride ||
                a.v[k][p].rhs_bytes != a.in[0].rhs_bytes)
                return false;
    }
    return true;
}
}  // namespace

hipError_t launch_wilson_mrhs(int sprec, int lprec, int recon, const WilsonArgs& args, int ny, int nrhs,
                              hipStream_t st) {
    WilsonArgs a = args;
    const MrhsShape sh = mrhs_shape(args.g, sprec, lprec, recon, nrhs, ny);
    a.order = make_order((a.g.vh + 63) / 64, a.g.n0, sh.chunk < 0 ? tile_order(a.g, 64) : sh.chunk);
    a.xcd_remap = sh.xcd_remap;
    MrhsGrid m;
    m.tiles = (a.g.vh + 63) / 64;
    m.ny = ny;
    m.rg = std::max(1, std::min(sh.rg > 0 ? sh.rg : nrhs, nrhs));
    m.ngroups = (nrhs + m.rg - 1) / m.rg;
    m.group_major = sh.group_major == 3 ? 1 : sh.group_major;   // 3 and no march: the tiles group-major
    m.nrhs = nrhs;
    m.per_part = 0;
    if (m.group_major == 2) {
        if (8 % m.ngroups != 0) {
            m.group_major = 1;   // XCD groups need a number of groups dividing 8
        } else {
            const int parts = 8 / m.ngroups;
            m.per_part = (int32_t)((m.tiles * (int64_t)ny + parts - 1) / parts);
        }
    }
    const int key = sprec * 1000 + lprec * 100 + recon;
    if (sh.group_major == 3 && march_fits(a, sprec, ny, nrhs)) {
        switch (lprec * 100 + recon) {
            case P32 * 100 + 18: return launch_march<P32, 18>(a, nrhs, st);
            case P32 * 100 + 12: return launch_march<P32, 12>(a, nrhs, st);
            case P32 * 100 + 8: return launch_march<P32, 8>(a, nrhs, st);
            case P16 * 100 + 18: return launch_march<P16, 18>(a, nrhs, st);
            case P16 * 100 + 12: return launch_march<P16, 12>(a, nrhs, st);
            default: return hipErrorInvalidValue;
        }
    }
    switch (key) {
        case P64 * 1000 + P64 * 100 + 18: return launch_mrhs_fmt<P64, P64, 18>(a, m, sh.link_nt, st);
        case P64 * 1000 + P64 * 100 + 12: return launch_mrhs_fmt<P64, P64, 12>(a, m, sh.link_nt, st);
        case P64 * 1000 + P64 * 100 + 8: return launch_mrhs_fmt<P64, P64, 8>(a, m, sh.link_nt, st);
        case P32 * 1000 + P32 * 100 + 18: return launch_mrhs_fmt<P32, P32, 18>(a, m, sh.link_nt, st);
        case P32 * 1000 + P32 * 100 + 12: return launch_mrhs_fmt<P32, P32, 12>(a, m, sh.link_nt, st);
        case P32 * 1000 + P32 * 100 + 8: return launch_mrhs_fmt<P32, P32, 8>(a, m, sh.link_nt, st);
        case P32 * 1000 + P16 * 100 + 18: return launch_mrhs_fmt<P32, P16, 18>(a, m, sh.link_nt, st);
        case P32 * 1000 + P16 * 100 + 12: return launch_mrhs_fmt<P32, P16, 12>(a, m, sh.link_nt, st);
        case P16 * 1000 + P32 * 100 + 18: return launch_mrhs_fmt<P16, P32, 18>(a, m, sh.link_nt, st);
        case P16 * 1000 + P32 * 100 + 12: return launch_mrhs_fmt<P16, P32, 12>(a, m, sh.link_nt, st);
        case P16 * 1000 + P32 * 100 + 8: return launch_mrhs_fmt<P16, P32, 8>(a, m, sh.link_nt, st);
        case P16 * 1000 + P16 * 100 + 18: return launch_mrhs_fmt<P16, P16, 18>(a, m, sh.link_nt, st);
        case P16 * 1000 + P16 * 100 + 12: return launch_mrhs_fmt<P16, P16, 12>(a, m, sh.link_nt, st);
        default: return hipErrorInvalidValue;
    }
}

int multi_grid_factor() { return g_multi_grid.load(std::memory_order_relaxed); }
void set_multi_grid_factor(int f) { g_multi_grid.store(f, std::memory_order_relaxed); }

hipError_t launch_wilson_multi(int sprec, int lprec, int recon, const MultiArgs& a, hipStream_t st) {
    const int key = sprec * 1000 + lprec * 100 + recon;
    switch (key) {
        case P64 * 1000 + P64 * 100 + 18: return launch_multi_fmt<P64, P64, 18>(a, st);
        case P64 * 1000 + P64 * 100 + 12: return launch_multi_fmt<P64, P64, 12>(a, st);
        case P64 * 1000 + P64 * 100 + 8: return launch_multi_fmt<P64, P64, 8>(a, st);
        case P32 * 1000 + P32 * 100 + 18: return launch_multi_fmt<P32, P32, 18>(a, st);
        case P32 * 1000 + P32 * 100 + 12: return launch_multi_fmt<P32, P32, 12>(a, st);
        case P32 * 1000 + P32 * 100 + 8: return launch_multi_fmt<P32, P32, 8>(a, st);
        case P32 * 1000 + P16 * 100 + 18: return launch_multi_fmt<P32, P16, 18>(a, st);
        case P32 * 1000 + P16 * 100 + 12: return launch_multi_fmt<P32, P16, 12>(a, st);
        case P16 * 1000 + P32 * 100 + 18: return launch_multi_fmt<P16, P32, 18>(a, st);
        case P16 * 1000 + P32 * 100 + 12: return launch_multi_fmt<P16, P32, 12>(a, st);
        case P16 * 1000 + P32 * 100 + 8: return launch_multi_fmt<P16, P32, 8>(a, st);
        case P16 * 1000 + P16 * 100 + 18: return launch_multi_fmt<P16, P16, 18>(a, st);
        case P16 * 1000 + P16 * 100 + 12: return launch_multi_fmt<P16, P16, 12>(a, st);
        default: return hipErrorInvalidValue;
    }
}

int march_slices(int n0, int64_t columns, int resident) {
    int best = n0;
    int64_t cost = INT64_MAX;
    // k rounds of `resident` workgroups hold seg segments of each column, so T is at
    // least n0 / seg; no k rounds cost less than the slices shared out evenly and 3 k
    for (int64_t k = (columns + resident - 1) / resident;; ++k) {
        if (cost < INT64_MAX && (2 * columns * n0 + resident - 1) / resident + 3 * k > cost) break;
        const int64_t seg = std::min<int64_t>(n0, k * resident / columns);
        const int T = (int)((n0 + seg - 1) / seg);
        const int64_t rounds = (columns * ((n0 + T - 1) / T) + resident - 1) / resident;
        const int64_t c = rounds * (2 * (int64_t)T + 3);
        if (c <= cost) {
            cost = c;
            best = T;
        }
        if (T == 1) break;
    }
    return best;
}

TileOrder make_order(int64_t tiles, int n0, int c) {
    TileOrder o;
    memset(&o, 0, sizeof(o));
    if (c <= 0) return o;
    o.c = c;
    o.cn = c * n0;
    o.slice = (int32_t)(tiles / n0);
    o.d_c = make_fastdiv((uint32_t)c);
    o.d_cn = make_fastdiv((uint32_t)o.cn);
    return o;
}

int tile_order(const GeomK& g, int block) {
    const int64_t per_slice = g.vh / g.n0;
    if (g.n0 < 4 || per_slice * g.n0 != g.vh || per_slice % block) return 0;
    const int64_t S = per_slice / block;
    const int64_t s1t = (g.s1 + block - 1) / block;   // x1 neighbours, in tiles
    for (int64_t c = std::max<int64_t>(2, 4 * s1t); c < S; ++c)
        if (S % c == 0) return (int)c;
    return 0;
}

WilsonArgs wilson_args(const ndq_geom* g, const ndq_gauge* U, int sprec) {
    WilsonArgs a;
    memset(&a, 0, sizeof(a));
    a.g = g->k;
    a.links = static_cast<const char*>(U->data);
    a.c0 = {1.0, nullptr};
    a.xcd_remap = tuning(sprec, U->prec, U->recon).xcd_remap;
    return a;
}

}  // namespace ndq

extern "C" {

int ndq_apply_Q(const ndq_geom* g, const ndq_gauge* U, double m, const ndq_spinor* in, const ndq_spinor* out,
                void* stream) {
    if (!g) return fail(NDQ_EINVAL, "ndq_apply_Q: NULL geometry");
    int rc = check_gauge(U);
    if (!rc) rc = check_spinor(g, in, NDQ_FULL, "ndq_apply_Q in");
    if (!rc) rc = check_spinor(g, out, NDQ_FULL, "ndq_apply_Q out");
    if (!rc) rc = check_pair(U, in);
    if (rc) return rc;
    if (in->prec != out->prec || in->nrhs != out->nrhs)
        return fail(NDQ_EINVAL, "ndq_apply_Q: in and out must share precision and nrhs");
    if (in->data == out->data) return fail(NDQ_EINVAL, "ndq_apply_Q: in and out must not alias");
    hipStream_t st = as_stream(stream);
    const bool batched = in->nrhs > 1;
    for (int r = 0; r < (batched ? 1 : in->nrhs); ++r) {
        WilsonArgs a = wilson_args(g, U, in->prec);
        a.p0 = 0;
        for (int p = 0; p < 2; ++p) {
            a.in[p] = view_of(g, in, 1 - p, r);
            a.self[p] = view_of(g, in, p, r);
            a.out[p] = view_of(g, out, p, r);
        }
        a.has_self = 1;
        a.a_self = 4.0 + m;
        a.b_hop = -0.5;
        a.gamma5 = 1;
        if (batched) NDQ_HIP(launch_wilson_mrhs(in->prec, U->prec, U->recon, a, 2, in->nrhs, st));
        else NDQ_HIP(launch_wilson(in->prec, U->prec, U->recon, a, 2, -1, st));
    }
    return NDQ_OK;
}

int ndq_apply_Q_multi(const ndq_q_job* jobs, int32_t njobs, void* stream) {
    if (!jobs || njobs < 1 || njobs > kMaxJobs)
        return fail(NDQ_EINVAL, "ndq_apply_Q_multi: need 1..%d jobs (got %d)", kMaxJobs, njobs);
    MultiArgs a;
    memset(&a, 0, sizeof(a));
    a.njobs = njobs;
    int64_t total = 0;
    int sprec = -1, lprec = -1, recon = -1;
    for (int j = 0; j < njobs; ++j) {
        const ndq_q_job& J = jobs[j];
        if (!J.g) return fail(NDQ_EINVAL, "ndq_apply_Q_multi: job %d: NULL geometry", j);
        int rc = check_gauge(J.U);
        if (!rc) rc = check_spinor(J.g, J.in, NDQ_FULL, "ndq_apply_Q_multi in");
        if (!rc) rc = check_spinor(J.g, J.out, NDQ_FULL, "ndq_apply_Q_multi out");
        if (!rc) rc = check_pair(J.U, J.in);
        if (rc) return rc;
        if (J.in->prec != J.out->prec || J.in->nrhs != J.out->nrhs)
            return fail(NDQ_EINVAL, "ndq_apply_Q_multi: job %d: in and out must share precision and nrhs", j);
        if (J.in->data == J.out->data) return fail(NDQ_EINVAL, "ndq_apply_Q_multi: job %d: in and out alias", j);
        if (j == 0) {
            sprec = J.in->prec;
            lprec = J.U->prec;
            recon = J.U->recon;
        } else if (J.in->prec != sprec || J.U->prec != lprec || J.U->recon != recon) {
            return fail(NDQ_EINVAL, "ndq_apply_Q_multi: job %d: all jobs must share spinor precision and link format", j);
        }
        QJob& q = a.job[j];
        q.g = J.g->k;
        q.links = static_cast<const char*>(J.U->data);
        for (int p = 0; p < 2; ++p) {
            q.in[p] = view_of(J.g, J.in, 1 - p, 0);
            q.self[p] = view_of(J.g, J.in, p, 0);
            q.out[p] = view_of(J.g, J.out, p, 0);
        }
        q.a_self = 4.0 + J.m;
        q.nrhs = J.in->nrhs;
        q.tiles = (J.g->vh + 63) / 64;
        q.tile0 = (int)total;
        total += 2 * (int64_t)q.tiles;
    }
    if (total > INT32_MAX) return fail(NDQ_EINVAL, "ndq_apply_Q_multi: too many sites");
    a.total = (int)total;
    NDQ_HIP(launch_wilson_multi(sprec, lprec, recon, a, as_stream(stream)));
    return NDQ_OK;
}

int ndq_apply_dslash(const ndq_geom* g, const ndq_gauge* U, const ndq_spinor* in, const ndq_spinor* out,
                     void* stream) {
    if (!g) return fail(NDQ_EINVAL, "ndq_apply_dslash: NULL geometry");
    int rc = check_gauge(U);
    if (!rc) rc = check_spinor(g, in, -1, "ndq_apply_dslash in");
    if (!rc) rc = check_spinor(g, out, -1, "ndq_apply_dslash out");
    if (!rc) rc = check_pair(U, in);
    if (rc) return rc;
    if (in->parity == NDQ_FULL || out->parity == NDQ_FULL || in->parity == out->parity)
        return fail(NDQ_EINVAL, "ndq_apply_dslash: in and out must be opposite parity fields");
    if (in->prec != out->prec || in->nrhs != out->nrhs)
        return fail(NDQ_EINVAL, "ndq_apply_dslash: in and out must share precision and nrhs");
    hipStream_t st = as_stream(stream);
    const int p = out->parity;
    const bool batched = in->nrhs > 1;
    for (int r = 0; r < (batched ? 1 : in->nrhs); ++r) {
        WilsonArgs a = wilson_args(g, U, in->prec);
        a.p0 = p;
        a.in[0] = view_of(g, in, 1 - p, r);
        a.out[0] = view_of(g, out, p, r);
        a.has_self = 0;
        a.b_hop = 1.0;
        a.gamma5 = 0;
        if (batched) NDQ_HIP(launch_wilson_mrhs(in->prec, U->prec, U->recon, a, 1, in->nrhs, st));
        else NDQ_HIP(launch_wilson(in->prec, U->prec, U->recon, a, 1, -1, st));
    }
    return NDQ_OK;
}

int ndq_apply_Qhat_ee(const ndq_geom* g, const ndq_gauge* U, double m, const ndq_spinor* in, const ndq_spinor* out,
                      const ndq_spinor* tmp, void* stream) {
    if (!g) return fail(NDQ_EINVAL, "ndq_apply_Qhat_ee: NULL geometry");
    int rc = check_gauge(U);
    if (!rc) rc = check_spinor(g, in, NDQ_EVEN, "ndq_apply_Qhat_ee in");
    if (!rc) rc = check_spinor(g, out, NDQ_EVEN, "ndq_apply_Qhat_ee out");
    if (!rc) rc = check_spinor(g, tmp, NDQ_ODD, "ndq_apply_Qhat_ee tmp");
    if (!rc) rc = check_pair(U, in);
    if (rc) return rc;
    if (in->prec != out->prec || in->prec != tmp->prec || in->nrhs != out->nrhs || tmp->nrhs < in->nrhs)
        return fail(NDQ_EINVAL, "ndq_apply_Qhat_ee: fields must share precision and nrhs");
    if (in->data == out->data) return fail(NDQ_EINVAL, "ndq_apply_Qhat_ee: in and out must not alias");
    if (4.0 + m == 0.0) return fail(NDQ_ESINGULAR, "ndq_apply_Qhat_ee: 4 + m = 0");
    hipStream_t st = as_stream(stream);
    for (int r = 0; r < in->nrhs; ++r) {
        WilsonArgs a = wilson_args(g, U, in->prec);
        a.p0 = 1;
        a.in[0] = view_of(g, in, 0, r);
        a.out[0] = view_of(g, tmp, 1, r);
        a.b_hop = 1.0;
        NDQ_HIP(launch_wilson(in->prec, U->prec, U->recon, a, 1, -1, st));
        WilsonArgs b = wilson_args(g, U, in->prec);
        b.p0 = 0;
        b.in[0] = view_of(g, tmp, 1, r);
        b.self[0] = view_of(g, in, 0, r);
        b.out[0] = view_of(g, out, 0, r);
        b.has_self = 1;
        b.a_self = 4.0 + m;
        b.b_hop = -1.0 / (4.0 * (4.0 + m));
        b.gamma5 = 1;
        NDQ_HIP(launch_wilson(in->prec, U->prec, U->recon, b, 1, -1, st));
    }
    return NDQ_OK;
}

}  // extern "C"

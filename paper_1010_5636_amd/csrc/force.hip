// Derivatives of y = Q[U] psi (Q of Sec. 2.1, Eq. 1) for a cotangent g.
//
// For a real function L of y with dL = Re<g, dy>, and links perturbed along su(3)
// as U_mu(x) -> exp(i w T_a) U_mu(x) (T_a = lambda_a / 2):
//
//   dL/dw^a_mu(x) = 1/2 Im tr(T_a G),
//   G = U_mu(x) H - K U_mu(x)^H,
//   H_ba = sum_s [(1 - gamma_mu) psi(x + mu)]_{s b} conj(chi(x)_{s a}),
//   K_ba = sum_s [(1 + gamma_mu) psi(x)]_{s b} conj(chi(x + mu)_{s a}),   chi = gamma5 g,
//
// because U_mu(x) enters D_W through the forward hop at x and the backward hop
// at x + mu, each with weight -1/2.  The gradient with respect to the complex
// link tensor in the tangent space is then 2 i sum_a F^a T_a U_mu(x), which
// satisfies Re<grad, i w T_a U> = w F^a.  One lane per (site, mu); FP64.
#include "ndq_internal.h"

using namespace ndq;

namespace {

// Upper two spins of (1 -+ gamma_mu) s with the chiral gamma matrices, as the
// stencil's hop functions project.  (1 -+ gamma_mu) is twice a projector, so
// <chi, (1 -+ gamma_mu) psi> = 1/2 <(1 -+ gamma_mu) chi, (1 -+ gamma_mu) psi>, and
// the lower spins of both factors repeat the upper ones: the colour matrices H and
// K are sums over two spins of these.
template <int MU, bool MINUS>
__device__ __forceinline__ void spin_project(const C<double> s[12], C<double> h[6]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const C<double> s0 = s[c], s1 = s[3 + c], s2 = s[6 + c], s3 = s[9 + c];
        C<double> a, b;   // h0 = s0 +- a, h1 = s1 +- b
        if constexpr (MU == 0) {
            a = s2;
            b = s3;
        } else if constexpr (MU == 1) {
            a = cmuli(s3);
            b = cmuli(s2);
        } else if constexpr (MU == 2) {
            a = s3;
            b = cneg(s2);
        } else {
            a = cmuli(s2);
            b = cmulmi(s3);
        }
        h[c] = MINUS ? cadd(s0, a) : csub(s0, a);
        h[3 + c] = MINUS ? cadd(s1, b) : csub(s1, b);
    }
}

// O_ba = sum over the two upper spins of p_{s b} conj(q_{s a})
__device__ __forceinline__ void outer(const C<double> p[6], const C<double> q[6], C<double> o[3][3]) {
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) o[b][a] = cfmac(cmulc(q[a], p[b]), q[3 + a], p[3 + b]);
}

struct ForceArgs {
    GeomK g;
    const char* links;
    SpinorView psi[2];   // parity views of psi
    SpinorView gv[2];    // parity views of g
    double* force;       // [V][4][8] (lexicographic) or nullptr
    double2* grad;       // [V][4][3][3] complex (lexicographic) or nullptr
};

constexpr double is3 = 0.57735026918962576451;   // 1/sqrt(3)

// U_mu(x) and its force components for the site (p, i) with neighbour nbr = x + mu.
template <int RECON, int MU>
__device__ __forceinline__ void link_force(const ForceArgs& a, int p, int32_t i, int32_t nbr, C<double> u[3][3],
                                           double f[8]) {
    C<double> H[3][3], K[3][3], G[3][3];
    {
        C<double> s[12], c[12], ps[6], pc[6];
        SpinorIO<P64>::load(a.psi[1 - p], (int64_t)a.psi[1 - p].site0 + nbr, s);
        SpinorIO<P64>::load(a.gv[p], (int64_t)a.gv[p].site0 + i, c);
#pragma unroll
        for (int k = 6; k < 12; ++k) c[k] = cneg(c[k]);   // chi = gamma5 g
        spin_project<MU, true>(s, ps);    // (1 - gamma_mu) psi(x + mu)
        spin_project<MU, true>(c, pc);    // (1 - gamma_mu) chi(x)
        outer(ps, pc, H);
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(H[b][k].r), "+v"(H[b][k].i));
    }
    __builtin_amdgcn_sched_barrier(0);   // not all 57 loads at once: their registers halve the wavefronts in flight
    {
        C<double> s[12], c[12], ps[6], pc[6];
        SpinorIO<P64>::load(a.psi[p], (int64_t)a.psi[p].site0 + i, s);
        SpinorIO<P64>::load(a.gv[1 - p], (int64_t)a.gv[1 - p].site0 + nbr, c);
#pragma unroll
        for (int k = 6; k < 12; ++k) c[k] = cneg(c[k]);
        spin_project<MU, false>(s, ps);   // (1 + gamma_mu) psi(x)
        spin_project<MU, false>(c, pc);   // (1 + gamma_mu) chi(x + mu)
        outer(ps, pc, K);
    }
    link_load<P64, RECON>(a.links, a.g.vh, p * 4 + MU, i, u);
    // G = U H - K U^H
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            C<double> acc = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc = cfma(acc, u[r][k], H[k][c]);
                acc = csub(acc, cmul(K[r][k], cconj(u[c][k])));
            }
            G[r][c] = acc;
        }
    // F^a = 1/2 Im tr(T_a G), T_a = lambda_a / 2 (Gell-Mann)
    f[0] = 0.25 * (G[1][0].i + G[0][1].i);                       // lambda_1: (0,1),(1,0) = 1
    f[1] = 0.25 * (G[0][1].r - G[1][0].r);                       // lambda_2: (0,1) = -i, (1,0) = i
    f[2] = 0.25 * (G[0][0].i - G[1][1].i);                       // lambda_3
    f[3] = 0.25 * (G[2][0].i + G[0][2].i);                       // lambda_4
    f[4] = 0.25 * (G[0][2].r - G[2][0].r);                       // lambda_5
    f[5] = 0.25 * (G[2][1].i + G[1][2].i);                       // lambda_6
    f[6] = 0.25 * (G[1][2].r - G[2][1].r);                       // lambda_7
    f[7] = 0.25 * is3 * (G[0][0].i + G[1][1].i - 2.0 * G[2][2].i);  // lambda_8
}

// One workgroup per 64 sites of one parity; wavefront w takes direction mu = w,
// so the four directions of a site read psi(x) and g(x) from the same cache
// lines at about the same time.  A site's outputs are 576 (gradient) and 256
// (force) contiguous bytes from four wavefronts: they meet in LDS and leave as
// whole lines.  Bound by HBM: 1216 bytes per site with 18-real links and the
// force, 1536 with the gradient; the gradient on 16^3x32 61 us with each lane
// storing its own 16-byte words and full four-spin products, 55 us here.
template <int RECON>
__global__ void __launch_bounds__(256) k_force(ForceArgs a) {
    constexpr int kRow = 37;   // double2 per site: 36 and one that spreads the banks
    __shared__ double2 out[64 * kRow];
    __shared__ int32_t site_lex[64];
    const int p = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t it = blockIdx.x * 64 + lane;
    const bool active = it < a.g.vh;
    const int32_t i = active ? it : a.g.vh - 1;   // lanes past the end repeat the last site and store nothing
    const int nsites = min(64, a.g.vh - (int32_t)blockIdx.x * 64);
    const SiteCoord x = eo_coords(a.g, p, i);
    int32_t nb[8];
    eo_neighbours(a.g, i, x, nb);
    C<double> u[3][3];
    double f[8];
    switch (mu) {
        case 0: link_force<RECON, 0>(a, p, i, nb[0], u, f); break;
        case 1: link_force<RECON, 1>(a, p, i, nb[1], u, f); break;
        case 2: link_force<RECON, 2>(a, p, i, nb[2], u, f); break;
        default: link_force<RECON, 3>(a, p, i, nb[3], u, f); break;
    }
    if (mu == 0) site_lex[lane] = 2 * i + (x.x3 & 1);
    if (a.force) {
        double* row = reinterpret_cast<double*>(out + lane * kRow) + mu * 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) row[k] = f[k];
        __syncthreads();
        // by doubles: the caller's array need not be aligned to more
        for (int e = threadIdx.x; e < nsites * 32; e += 256)
            a.force[(int64_t)site_lex[e >> 5] * 32 + (e & 31)] =
                reinterpret_cast<const double*>(out + (e >> 5) * kRow)[e & 31];
        if (a.grad) __syncthreads();   // before the gradient takes the rows
    }
    if (a.grad) {
        // 2 i sum_a f_a T_a U = i (sum_a f_a lambda_a) U
        C<double> Lm[3][3];
        Lm[0][0] = {f[2] + is3 * f[7], 0.0};
        Lm[1][1] = {-f[2] + is3 * f[7], 0.0};
        Lm[2][2] = {-2.0 * is3 * f[7], 0.0};
        Lm[0][1] = {f[0], -f[1]};
        Lm[1][0] = {f[0], f[1]};
        Lm[0][2] = {f[3], -f[4]};
        Lm[2][0] = {f[3], f[4]};
        Lm[1][2] = {f[5], -f[6]};
        Lm[2][1] = {f[5], f[6]};
        double2* row = out + lane * kRow + mu * 9;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                C<double> acc = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) acc = cfma(acc, Lm[r][k], u[k][c]);
                const C<double> v = cmuli(acc);
                row[3 * r + c] = make_double2(v.r, v.i);
            }
        __syncthreads();
        for (int e = threadIdx.x; e < nsites * 36; e += 256) {
            const int s = e / 36, k = e - 36 * s;
            a.grad[(int64_t)site_lex[s] * 36 + k] = out[s * kRow + k];
        }
    }
}

}  // namespace

extern "C" int ndq_gauge_force(const ndq_geom* g, const ndq_gauge* U, const ndq_spinor* psi, const ndq_spinor* gy,
                               double* d_force, void* d_grad, void* stream) {
    if (!g) return fail(NDQ_EINVAL, "ndq_gauge_force: NULL geometry");
    int rc = check_gauge(U);
    if (!rc) rc = check_spinor(g, psi, NDQ_FULL, "ndq_gauge_force psi");
    if (!rc) rc = check_spinor(g, gy, NDQ_FULL, "ndq_gauge_force g");
    if (rc) return rc;
    if (U->prec != NDQ_F64 || psi->prec != NDQ_F64 || gy->prec != NDQ_F64)
        return fail(NDQ_EPREC, "ndq_gauge_force: FP64 links and spinors");
    if (psi->nrhs != 1 || gy->nrhs != 1) return fail(NDQ_EINVAL, "ndq_gauge_force: one right-hand side");
    if (!d_force && !d_grad) return fail(NDQ_EINVAL, "ndq_gauge_force: no output requested");
    ForceArgs a;
    a.g = g->k;
    a.links = static_cast<const char*>(U->data);
    for (int p = 0; p < 2; ++p) {
        a.psi[p] = view_of(g, psi, p, 0);
        a.gv[p] = view_of(g, gy, p, 0);
    }
    a.force = d_force;
    a.grad = static_cast<double2*>(d_grad);
    const dim3 grid((g->vh + 63) / 64, 2);
    hipStream_t st = as_stream(stream);
    switch (U->recon) {
        case 18: hipLaunchKernelGGL(k_force<18>, grid, dim3(256), 0, st, a); break;
        case 12: hipLaunchKernelGGL(k_force<12>, grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL(k_force<8>, grid, dim3(256), 0, st, a); break;
    }
    NDQ_HIP(hipGetLastError());
    return NDQ_OK;
}

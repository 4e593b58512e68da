// P2G on gfx950: particle-to-grid transfer with the deferred deformation
// update, the snow return map and the Kirchhoff stress fused in (paper,
// "Merge Kernels": plasticity, SVD and stress computed inside P2G).
//
// Avoiding non-native intrinsics ("Avoid non-native intrinsics"): on V100
// the paper drops shared-memory float atomics because they are emulated.
// On gfx950 ds_add_f32 exists but runs at about 0.3 lane-ops per clock per
// CU, while ds_add_f64 runs at about 6.6 and ds_add_u64 at 9.1 (and far
// better under bank and address conflicts), and global float atomics (about
// 0.4, executed memory-side) move a full write per update.  The same
// principle -- use only the fast native operations -- leads here to:
//   * a workgroup takes one chunk (<= 256 or 512 particles of one particle
//     block), one particle per thread, loads coalesced;
//   * phase 1 computes every particle's contribution and the bounding box of
//     the stencils of the chunk's in-zone particles (block reduction);
//   * the tile is that box (at most 1024 padded nodes; a particle block's
//     stencils cover 6^3 = 216 nodes right after a rebuild), four 64-bit
//     fixed-point channels (weight sum and three momentum components, the
//     latter scaled per chunk) accumulated with ds_add_u64: exact, so the
//     sums do not depend on the order of the adds;
//   * the tile is then STORED (plain, coalesced float4 stores) to the
//     staging buffer; the rebuild registered each chunk with every physical
//     block its in-zone stencils can reach, and the grid update gathers each
//     node from the registered tiles whose box holds it, in chunk order --
//     no global atomics, and the transfer of in-zone particles is
//     deterministic.  Each workgroup owns an
//     equal slice of the staging buffer and packs its chunks' tiles there
//     (offset recorded per chunk), so no allocation is shared.
// The rebuild stores each chunk dealt over its 16-lane LDS passes by the
// bank pair of each particle's cell in this tile layout, so the 16 lanes of
// one LDS access meet each bank pair about as rarely as the chunk's cells
// allow and rarely share an address (conflicting lanes of a pass
// serialize; lanes in different passes do not conflict).
// Particles outside their free zone (before a late rebuild) scatter straight
// to global atomics and activate the blocks they touch.
#include <type_traits>

#include "mpm_kernels.h"
#include "mpm_mlp.h"

namespace mpm {

namespace {

constexpr int CT = 1024;  // LDS tile capacity in nodes (padded layout, below)

// LDS tile layout: the padded node-box layout (pitch_row, pitch_plane in
// mpm_kernels.h), four 64-bit fixed-point channels: the weight sum in units
// of 2^-FRAC_W and the three momentum components in units of 2^-FRAC_M of the
// chunk's momentum scale (below).  Integer adds are exact and
// order-independent, and ds_add_u64 meets far fewer conflict cycles than
// ds_add_f64 (a replay of late-frame snow stencils: 14 against 22 cycles per
// wave instruction).
//
// A contribution becomes a fixed-point word in one FP64 multiplication: the
// bits of a non-negative denormal k 2^-1074 are the integer k (and up to
// 2^53, where the exponent field becomes 1, they go on counting), so a product
// scaled into that range comes out rounded to the nearest unit, as a 64-bit
// integer.  Momentum is made non-negative by adding the chunk's bound K to
// it (w (m + K) instead of w m); the tile store takes K times the weight sum
// off again.  FP64 keeps denormals in every build (the flush-to-zero of the
// fast-math build is FP32's).  About 10 instructions per node and particle,
// against 20 with FP32 products, a conversion, a rounding addition and a
// subtraction of its bits per channel (and 24, with a branch per node, in the
// 59% of the waves that tested every term for a tiny weight): VALU issue binds
// this kernel at scenes of a million particles (84% busy before), the longest
// workgroup at small ones.  Fused P2G before and after: 109.6 -> 101.6 us on
// snow of 1.39M particles, 259 -> 244 us on sand of 3.1M, 16.5 -> 14.4 us on
// jelly of 32K (96.5, 228 and 11.5 to 12.2 with what else has changed since).
constexpr int FRAC_W = 54;  // weight: w <= 27/64, below 2^53 units; 512 of them below 2^62
constexpr int FRAC_M = 53;  // momentum: w (m + K) scaled below 2^53 units
constexpr double DENORM_SPLIT = 0x1p-1000;  // the weights' share of the scale into the denormal range
// A weight below LIGHT_W (2^-32) is resolved to too few units by itself, and
// the roundings of many such terms need not cancel (a plane of particles just
// beyond a cell edge: all equal).  A node of the tile that holds some is good
// to a few FP32 roundings all the same where its weight sum is at least 2^-33
// for each of the chunk's L particles that have such a weight anywhere in
// their stencil: its light terms, good to half a unit each, are then off by
// 2^-22 of the sum together, its others by 2^-23 of themselves.  A node below
// that (L << WEAK_SHIFT units) is weak: the tile store lists it, and its
// particles add to it again, in FP64 and unscaled.  About one particle in 70
// has a light weight (59% of the waves), but only a node at the very edge of a
// chunk's material has no other contribution: without light particles no node
// is weak, with the usual four of a chunk few are (runs of 32K to 3.1M
// particles take 0.0% to 0.5% longer than with one unit added to every term
// and a bound of 2^-32 for any L, which left equal terms' roundings at up to
// 9e-5 of a node's mass).
// One particle in 4 10^4 has a weight that may round to nothing: it adds one
// unit more to its nodes, so that a node that only such weights reach shows
// (were all L such particles, 2^-21 of the sum).
constexpr float LIGHT_W = 0x1.01p-32f;  // (with room for the rounding of a product of FP32 weights)
constexpr int WEAK_SHIFT = FRAC_W - 33;

// Contexts with an ASFLIP scene keep FP32 terms (F32 below), whatever map
// their snow scenes take: the products w and w m are rounded to FP32, then to
// units of 2^-51 (weight) and 2^(em - 50) (momentum) as two's complement
// words, and a term of weight below 2^-32 goes to the node's global
// accumulator.  ASFLIP's position share jumps where a particle's volume change
// crosses 1, so any other rounding of a node velocity sends some particles of
// a frame another way (of 142K fountain particles about 60 in 44 substeps, J
// then off by up to 2e-3): there results stay comparable from build to build
// only with the same rounding.  It costs about 2 us per launch.
constexpr float W_SCALE_F32 = 0x1p51f;
constexpr int FRAC_M_F32 = 50;
constexpr float TINY_W = 0x1p-32f;

// Round-to-nearest integer of y (|y| < 2^51) as a 64-bit two's-complement
// word: adding 1.5 2^52 in FP64 leaves the integer in the low mantissa bits.
__device__ __forceinline__ unsigned long long fixed64(float y) {
    return (unsigned long long)(__double_as_longlong((double)y + 0x1.8p52) - 0x4338000000000000LL);
}

__device__ __forceinline__ float pick3(const float w[3], int o) { return o == 0 ? w[0] : o == 1 ? w[1] : w[2]; }

// ------------------------------------------------ snow return map without SVD
// Eigenvalues of the symmetric b = [b0 b1 b2; . b3 b4; . . b5] as
// q + p mu_k, mu descending, by the trigonometric solution of the
// characteristic cubic of the normalised deviator Bn = (b - q I)/p (whose
// eigenvalues mu satisfy mu^3 - 3 mu - det Bn = 0).  Returns false when b is
// too close to a multiple of the identity for the deviator to be resolved.
__device__ __forceinline__ bool eig_closed(const float b[6], float& q, float& p, float mu[3], float Bn[6]) {
    q = (b[0] + b[3] + b[5]) * (1.0f / 3.0f);
    const float d0 = b[0] - q, d1 = b[3] - q, d2 = b[5] - q;
    const float p2 = d0 * d0 + d1 * d1 + d2 * d2 + 2.0f * (b[1] * b[1] + b[2] * b[2] + b[4] * b[4]);
    p = sqrtf(p2 * (1.0f / 6.0f));
    if (!(p > 2e-5f * fabsf(q))) return false;
    const float ip = 1.0f / p;
    Bn[0] = d0 * ip; Bn[1] = b[1] * ip; Bn[2] = b[2] * ip;
    Bn[3] = d1 * ip; Bn[4] = b[4] * ip; Bn[5] = d2 * ip;
    const float det = Bn[0] * (Bn[3] * Bn[5] - Bn[4] * Bn[4]) - Bn[1] * (Bn[1] * Bn[5] - Bn[4] * Bn[2]) +
                      Bn[2] * (Bn[1] * Bn[4] - Bn[3] * Bn[2]);
    const float phi = acosf(fminf(fmaxf(0.5f * det, -1.0f), 1.0f)) * (1.0f / 3.0f);
    mu[0] = 2.0f * cosf(phi);
    mu[2] = 2.0f * cosf(phi + 2.09439510f);  // + 2 pi / 3
    mu[1] = -mu[0] - mu[2];
    return true;
}

// sum_k c_k L_k(Bn) = A2 Bn^2 + A1 Bn + A0 I, with L_k the Lagrange
// polynomials on the (distinct) eigenvalues mu: each L_k(Bn) is the
// projector on eigenvector k (Sylvester's formula), so isotropic functions
// of b are built without eigenvectors.
__device__ __forceinline__ void lagrange(const float mu[3], const float c[3], float& A2, float& A1, float& A0) {
    A2 = A1 = A0 = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int i = (k + 1) % 3, j = (k + 2) % 3;
        const float w = c[k] / ((mu[k] - mu[i]) * (mu[k] - mu[j]));
        A2 += w;
        A1 += w * mu[k];  // -(mu_i + mu_j) = mu_k since the mu sum to zero
        A0 += w * mu[i] * mu[j];
    }
}

// The snow return map and Kirchhoff stress of every lane's particle from the
// eigenvalues of b = F^ F^T alone: F_E' = (I + sum_k delta_k L_k) F^ and
// tau = tau_bar I + sum_k (tau_k - tau_bar) L_k, with delta_k = s'_k/s_k - 1.
// The projected values come from the exact clamp (ret = 2) or from the
// network (ret = 1; all lanes of the wave run it on MFMA).  A lane falls
// back to the exact (Jacobi) map when its eigenvalues are too close, its
// particle is inverted, or (network) the prediction leaves the yield
// surface or changes the total volume by more than the tolerance.
template <bool NET>
__device__ void snow_without_svd(const mlp::NetLds16* net, float* stage, const Scenes& T, const Scene& sc, float dt,
                                 int pending, bool have, const float C[9], float F[9], float& s, float tau[6],
                                 bool& fell_back) {
    const Mat& M = sc.M;
    float Fh[9];
    if (pending) {
        advance_gradient(C, dt, F, Fh);
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) Fh[k] = F[k];
    }
    float b[6];
    b[0] = Fh[0] * Fh[0] + Fh[1] * Fh[1] + Fh[2] * Fh[2];
    b[1] = Fh[0] * Fh[3] + Fh[1] * Fh[4] + Fh[2] * Fh[5];
    b[2] = Fh[0] * Fh[6] + Fh[1] * Fh[7] + Fh[2] * Fh[8];
    b[3] = Fh[3] * Fh[3] + Fh[4] * Fh[4] + Fh[5] * Fh[5];
    b[4] = Fh[3] * Fh[6] + Fh[4] * Fh[7] + Fh[5] * Fh[8];
    b[5] = Fh[6] * Fh[6] + Fh[7] * Fh[7] + Fh[8] * Fh[8];
    float q, p, mu[3], Bn[6];
    bool use = have && eig_closed(b, q, p, mu, Bn) && det3(Fh) > 0.0f;
    use = use && (mu[0] - mu[1]) >= T.sur_gap && (mu[1] - mu[2]) >= T.sur_gap;
    float sh[3], sn[3], tk[3], Jpn;
#pragma unroll
    for (int k = 0; k < 3; ++k) sh[k] = use ? sqrtf(fmaxf(q + p * mu[k], 1e-30f)) : 1.0f;
    const float Jp = use ? s : 1.0f;
    if (NET && pending && __ballot(use) != 0ull) {  // a wave with no eligible lane skips the network
        // features [s, ln s, J_P, ln J_P, h, dt/dt_ref, s1 s2 s3, 1], the wave's 64 samples at once.
        // dt/dt_ref is exactly 1 at the training step (a refined division): a feature that was
        // constant in training has a floored spread (1e-6), so one ulp off would move its
        // normalised value by 0.06 and the J_P output by about 4e-4.
        const float dtr = div_refined(dt, T.sur_dt_ref);
        const float xf[SUR_IN] = {sh[0], sh[1], sh[2], logf(sh[0]), logf(sh[1]), logf(sh[2]), Jp, logf(Jp),
                                  expf(M.xi * (1.0f - Jp)), dtr, sh[0] * sh[1] * sh[2], 1.0f};
        float xn[SUR_IN], yv[SUR_OUT];
#pragma unroll
        for (int f = 0; f < SUR_IN; ++f) xn[f] = (xf[f] - net->imu[f]) / net->isd[f];
        mlp::forward_wave16(*net, stage, xn, yv);
#pragma unroll
        for (int o = 0; o < SUR_OUT; ++o) yv[o] = yv[o] * net->osd[o] + net->omu[o];
        // outputs [s', ln(s'/s), tau/E, J_P'/J_P, h', s1's2's3']: the projected state comes from
        // ln(s'/s) and J_P'/J_P; the stress is evaluated from that state, and the network's own
        // stress outputs serve as a consistency check
        float res_t = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) sn[k] = sh[k] * expf(yv[3 + k]);
        Jpn = Jp * yv[9];
        {
            const float h = expf(M.xi * (1.0f - Jpn));
            const float Jn = sn[0] * sn[1] * sn[2];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                tk[k] = 2.0f * M.mu * h * (sn[k] - 1.0f) * sn[k] + M.la * h * (Jn - 1.0f) * Jn;
                res_t = fmaxf(res_t, fabsf(yv[6 + k] - tk[k] / sc.E));
            }
        }
        float res_y = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) res_y = fmaxf(res_y, fmaxf(M.lo - sn[k], sn[k] - M.hi));
        const float res_v = fabsf(logf(sn[0] * sn[1] * sn[2] * Jpn) - logf(sh[0] * sh[1] * sh[2] * Jp));
        const bool fin = isfinite(tk[0] + tk[1] + tk[2] + Jpn + sn[0] + sn[1] + sn[2]);
        use = use && fin && res_y <= T.sur_tol && res_v <= T.sur_tol && res_t <= T.sur_tol;
    } else {
        // exact clamp; with nothing pending the stored state is already projected
        // (as in the exact path), so only the stress is evaluated
#pragma unroll
        for (int k = 0; k < 3; ++k) sn[k] = pending ? fminf(fmaxf(sh[k], M.lo), M.hi) : sh[k];
        Jpn = Jp * (sh[0] * sh[1] * sh[2]) / (sn[0] * sn[1] * sn[2]);
        const float h = expf(M.xi * (1.0f - Jpn));
        const float Jn = sn[0] * sn[1] * sn[2];
#pragma unroll
        for (int k = 0; k < 3; ++k) tk[k] = 2.0f * M.mu * h * (sn[k] - 1.0f) * sn[k] + M.la * h * (Jn - 1.0f) * Jn;
    }
    fell_back = have && !use;
    if (!have) return;
    if (!use) {
        material_step(M, dt, pending, C, F, s, tau);
        return;
    }
    float B2[6];
    B2[0] = Bn[0] * Bn[0] + Bn[1] * Bn[1] + Bn[2] * Bn[2];
    B2[1] = Bn[0] * Bn[1] + Bn[1] * Bn[3] + Bn[2] * Bn[4];
    B2[2] = Bn[0] * Bn[2] + Bn[1] * Bn[4] + Bn[2] * Bn[5];
    B2[3] = Bn[1] * Bn[1] + Bn[3] * Bn[3] + Bn[4] * Bn[4];
    B2[4] = Bn[1] * Bn[2] + Bn[3] * Bn[4] + Bn[4] * Bn[5];
    B2[5] = Bn[2] * Bn[2] + Bn[4] * Bn[4] + Bn[5] * Bn[5];
    // F_E' = G F^ with G = I + sum_k delta_k L_k
    float dl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) dl[k] = sn[k] / sh[k] - 1.0f;
    float A2, A1, A0;
    lagrange(mu, dl, A2, A1, A0);
    float G[6];
#pragma unroll
    for (int e = 0; e < 6; ++e) G[e] = A2 * B2[e] + A1 * Bn[e];
    G[0] += 1.0f + A0;
    G[3] += 1.0f + A0;
    G[5] += 1.0f + A0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float f0 = Fh[0 * 3 + c], f1 = Fh[1 * 3 + c], f2 = Fh[2 * 3 + c];
        F[0 * 3 + c] = G[0] * f0 + G[1] * f1 + G[2] * f2;
        F[1 * 3 + c] = G[1] * f0 + G[3] * f1 + G[4] * f2;
        F[2 * 3 + c] = G[2] * f0 + G[4] * f1 + G[5] * f2;
    }
    s = Jpn;
    // tau = tau_bar I + sum_k (tau_k - tau_bar) L_k
    const float tb = (tk[0] + tk[1] + tk[2]) * (1.0f / 3.0f);
    const float dt3[3] = {tk[0] - tb, tk[1] - tb, tk[2] - tb};
    lagrange(mu, dt3, A2, A1, A0);
#pragma unroll
    for (int e = 0; e < 6; ++e) tau[e] = A2 * B2[e] + A1 * Bn[e];
    tau[0] += tb + A0;
    tau[3] += tb + A0;
    tau[5] += tb + A0;
}

// NT threads per workgroup = the largest chunk it takes (128, 256 or 512).
// SURM: 0 every snow scene takes the exact map; 1 some scene takes the
// closed form without SVD; 2 some scene takes the network (staged in LDS).
// FUSED (with the tile path and the exact map only): each chunk first does
// the previous substep's G2P -- gathered from the node box of that
// substep's tile, staged in the tile's LDS -- and scatters with the fresh
// v, C and x; the particle's v and C are not stored (the G2P that brings the
// state up to date before a read recomputes them).  vel, host_flag and
// fb_limit serve that G2P.
template <bool GLOBAL_ONLY, int NT, int SURM, bool FUSED, bool F32 = false>
__device__ __forceinline__ void p2g_body(float* __restrict__ S, int64_t cap_, const Chunk* __restrict__ chunks,
                                         int* __restrict__ ctl, float* __restrict__ acc,
                                         int* __restrict__ acc_dirty, float4* __restrict__ stage,
                                         int stage_nodes, int4* __restrict__ box, int* __restrict__ brick_state,
                                         int* __restrict__ ovf, int parity, const Scenes& T, int pending,
                                         int nbricks, int act, const float4* __restrict__ vel,
                                         int* __restrict__ host_flag, int fb_limit) {
    static_assert(!F32 || (!GLOBAL_ONLY && !FUSED), "FP32 terms: the separate tile path");
    static_assert(!FUSED || (!GLOBAL_ONLY && SURM == 0), "the fused G2P needs the LDS tile and the exact map");
    __shared__ __align__(16) double tq[GLOBAL_ONLY ? 1 : 4 * CT];
    __shared__ int red_i[8][NT / 64];
    // weak nodes of the tile: their box coordinates, 5 bits an axis (a box spans at most 16 nodes:
    // the reach of one 2x2x1 slab of blocks)
    __shared__ unsigned short weak[GLOBAL_ONLY ? 1 : CT];
    __shared__ int n_weak;
#ifndef MPM_WEIGHTS_IN_LDS
#define MPM_WEIGHTS_IN_LDS 0
#endif
#if MPM_WEIGHTS_IN_LDS
    __shared__ float wpark[9 * NT];
#endif
    struct Empty {};
    __shared__ typename std::conditional<SURM == 2, mlp::NetLds16, Empty>::type net;
    __shared__ __attribute__((aligned(16))) float sur_stage[SURM == 2 ? NT / 64 * mlp::FWD_STAGE : 1];
    if constexpr (SURM == 2) {
        if (T.sur_theta) mlp::load_net16<NT>(net, T.sur_theta, T.sur_norm);
        __syncthreads();
    }
    int begin, end, stride;
    xcd_split(rank_limit(T, ctl, act, RE_CHUNK, CTL_NCHUNK), begin, end, stride);
    if constexpr (!GLOBAL_ONLY) {  // (workgroup-uniform: skipped by a workgroup without chunks)
        if (begin < end) {
            for (int t = threadIdx.x; t < 4 * CT; t += NT) tq[t] = 0.0;
            if (threadIdx.x == 0) n_weak = 0;
            __syncthreads();
        }
    }
    unsigned err = 0;
    unsigned n_sur = 0, n_fb = 0;
    // fused G2P: the free-zone request, made for particles that left and ahead
    // for a body that is about to (below; the G2P kernel's own request comes
    // after the exit only), and for tile fallbacks (the previous substep's P2G
    // counted them in the other slot)
    bool left = FUSED && blockIdx.x == 0 && threadIdx.x == 0 && ctl[CTL_FB + (parity ^ 1)] > fb_limit;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // this workgroup's slice of the staging buffer, filled front to back
    const int slice = (int)((int64_t)stage_nodes / gridDim.x);
    const int slice0 = slice * (int)blockIdx.x;
    int used = 0;
    for (int c = begin; c < end; c += stride) {
        int64_t cap = cap_;  // opaque per chunk: hoisted, the fields' 27 bases spill scalar registers
        asm("" : "+s"(cap));
        const Chunk ch = chunks[c];
        const Scene& sc = T.scene[ch.scene];
        Step P = sc.P;
        Mat M = sc.M;
        int brick_base = sc.brick_base;
        if constexpr (!FUSED) {
            // the words that branches and addresses wait for, through the scalar cache (no kernel writes the
            // table): ASFLIP water of 143K particles 21.9 -> 20.4 us; nothing for the fused kernel, whose
            // loads wait for its node box
            const auto* cs = (const __attribute__((address_space(4))) Scene*)(uintptr_t)&sc;
            P.n = cs->P.n;
            P.NB = cs->P.NB;
            M.kind = cs->M.kind;
            brick_base = cs->brick_base;
        }
        const int NB = P.NB;
        const float dx = P.dx, dt = P.dt;
        const int count = ch.count;
        const bool have = tid < count;
        const int p = ch.start + (have ? tid : 0);

        // ---- phase 1: material update, stress and this particle's payload
        Stencil st;
        float q[3] = {0.f, 0.f, 0.f}, Ad[9];
        bool ok = false, in_zone = false;
        // (lanes past the chunk's end load its first particle: no branch and no defaults)
        float x[3], v[3] = {0.f, 0.f, 0.f}, C[9], F[9], s, tau[6];
#pragma unroll
        for (int a = 0; a < 3; ++a) x[a] = field(S, FX + a, p, cap);
#pragma unroll
        for (int k = 0; k < 9; ++k) C[k] = FUSED ? 0.0f : field(S, FC + k, p, cap);
        if (!FUSED) {
#pragma unroll
            for (int a = 0; a < 3; ++a) v[a] = field(S, FV + a, p, cap);
        }
        s = field(S, FS, p, cap);
        int B[3];  // the particle's block at the last rebuild (its free zone)
        fsid_block(field(S, FSID, p, cap), B);
        if (M.kind != MPM_WATER) {
#pragma unroll
            for (int k = 0; k < 9; ++k) F[k] = field(S, FF + k, p, cap);
        } else {
#pragma unroll
            for (int k = 0; k < 9; ++k) F[k] = 0.0f;  // not used
        }
        int ng = 0, ngs = 0;  // fused G2P: nodes of the previous box, and the LDS float4 they span
        if constexpr (FUSED) {
            const int4 bb = box[c];
            const int lg[3] = {bb.x & 1023, (bb.x >> 10) & 1023, bb.x >> 20};
            const int eg[3] = {bb.y & 255, (bb.y >> 8) & 255, bb.y >> 16};
            ng = eg[0] * eg[1] * eg[2];
            const int Rg = pitch_row(eg[0]), Qg = pitch_plane(Rg, eg[1]);  // padded: no bank conflicts
            ngs = ng > 0 ? Qg * eg[2] : 0;
            if (ngs > 2 * CT) ng = ngs = 0;  // the tile holds 2 CT float4
            float4* tv = reinterpret_cast<float4*>(tq);
            const float4* vels = vel + (int64_t)brick_base * BLOCK_NODES;
            load_node_box(tv, vels, NB, lg, eg, ng, Rg, Qg, tid, NT);
            __syncthreads();
            Stencil sg;
            if (have && make_stencil(x, P, sg, err)) {
                g2p_gather(sg, tv, vels, NB, lg, eg, ng, Rg, Qg, 4.0f * P.fn, v, C);
                bool fin = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    x[a] += dt * v[a];
                    field(S, FX + a, p, cap) = x[a];
                    fin = fin && (fabsf(x[a]) < 1e30f) && (fabsf(v[a]) < 1e30f);
                }
                if (!fin) err |= MPM_ERR_NONFINITE;
            }
        }
        bool sur_chunk = false;
        if constexpr (SURM != 0) {
            sur_chunk = sc.ret != 0 && M.kind == MPM_SNOW;  // uniform over the workgroup
            if (sur_chunk) {
                bool fb = false;
                if constexpr (SURM == 2) {
                    if (sc.ret == 1)
                        snow_without_svd<true>(&net, sur_stage + wv * mlp::FWD_STAGE, T, sc, dt, pending, have, C, F, s, tau, fb);
                    else
                        snow_without_svd<false>(&net, sur_stage, T, sc, dt, pending, have, C, F, s, tau, fb);
                } else {  // no network in this variant
                    snow_without_svd<false>(nullptr, nullptr, T, sc, dt, pending, have, C, F, s, tau, fb);
                }
                n_sur += __popcll(__ballot(have && !fb));
                n_fb += __popcll(__ballot(fb));
            }
        }
        if (!sur_chunk && have) material_step(M, dt, pending, C, F, s, tau);
        if (have) {
            if (pending) {  // the deferred update of the last G2P lands here
                if (M.kind != MPM_WATER) {
#pragma unroll
                    for (int k = 0; k < 9; ++k) field(S, FF + k, p, cap) = F[k];
                }
                if (M.kind != MPM_JELLY) field(S, FS, p, cap) = s;
            }
            ok = make_stencil(x, P, st, err);
#if MPM_WEIGHTS_IN_LDS  // the register-pressure ablation: weights parked in LDS until the scatter
#pragma unroll
            for (int k = 0; k < 9; ++k) wpark[k * NT + tid] = st.w[k / 3][k % 3];
#endif
            // A = m C - (4 dt V0 / dx^2) tau;  Ad = dx A;  q = m v - Ad f, so the
            // momentum sent to stencil node o is w_o (q + Ad o).
            const float Tf[9] = {tau[0], tau[1], tau[2], tau[1], tau[3], tau[4], tau[2], tau[4], tau[5]};
#pragma unroll
            for (int k = 0; k < 9; ++k) Ad[k] = dx * (M.mp * C[k] - M.scale * Tf[k]);
#pragma unroll
            for (int a = 0; a < 3; ++a)
                q[a] = M.mp * v[a] - (Ad[a * 3 + 0] * st.f[0] + Ad[a * 3 + 1] * st.f[1] + Ad[a * 3 + 2] * st.f[2]);
            bool zone = true;  // the cell code base + 1 within the particle's free zone [4B-3, 4B+6]
#pragma unroll
            for (int a = 0; a < 3; ++a) zone = zone && (unsigned)(st.base[a] - (4 * B[a] - 4)) <= (unsigned)(TILE - 3);
            in_zone = ok && zone;
            if constexpr (FUSED) {
                left = left || (ok && !zone);  // (a particle outside the grid stays where it is)
                // A body that moves as one leaves its zone all at once, and the host sees the request some
                // substeps late: a wave of every eighth chunk asks AHEAD substeps early (the cadence at which
                // the host looks).  Sand of 3.1M, falling and splashing: 258.4 -> 252.5 us on average, the
                // longest launch 1080 -> 322, 24 -> 26 rebuilds in 828 substeps.  In every chunk the test
                // costs 0.4% to 0.8% where nothing leaves (snow, 64 scenes); so, nothing.
                constexpr float AHEAD = 4.0f;
                if (wv == 0 && (c & 7) == 0) {
                    bool stays = true;
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        const float y = (x[a] + (AHEAD * dt) * v[a]) * P.fn - 0.5f - (float)(4 * B[a] - 4);
                        stays = stays && y >= 0.0f && y < (float)(TILE - 2);
                    }
                    left = left || (ok && !stays);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < 9; ++k) Ad[k] = 0.0f;
        }

        // ---- the box of the in-zone stencils of the chunk
        int lo[3] = {0, 0, 0}, ext[3] = {0, 0, 0};
        int nt = 0, off = 0, R = 4, Q = 8;  // tight node count, staging offset, LDS pitches
        float m_bound = 0.0f;  // K, above every |m| of the chunk
        int em = 0;            // 27/64 (m + K) < 2^em: momentum units are 2^(em - FRAC_M)
        int copies = 1;        // of the tile, an odd number of nodes apart (different banks)
        float wmin = 1.0f;     // the smallest weight of the particle's stencil
        int lights = 0;        // the chunk's particles with a weight below LIGHT_W
        // the smallest of a stencil's 27 weights is the product of its per-axis minima
        auto smallest_weight = [&] {
            float w = 1.0f;
#pragma unroll
            for (int a = 0; a < 3; ++a) w *= fminf(fminf(st.w[a][0], st.w[a][1]), st.w[a][2]);
            return w;
        };
        if (GLOBAL_ONLY && tid == 0) box[c] = make_int4(0, 0, 0, 0);
        if (!GLOBAL_ONLY) {
            const bool in_tile = have && in_zone;
            int mn[3], mx[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                mn[a] = wave_min(in_tile ? st.base[a] : INT_MAX);
                mx[a] = wave_max(in_tile ? st.base[a] + 2 : INT_MIN);
            }
            // bound on |q_a + Ad_a . o| over the stencil (o in {0,1,2}^3), the momentum a tiled
            // particle sends to a node before its weight (non-negative: ordered as an int)
            float mb = 0.0f;
            if (in_tile) {
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    mb = fmaxf(mb, fabsf(q[a]) + 2.0f * (fabsf(Ad[3 * a]) + fabsf(Ad[3 * a + 1]) + fabsf(Ad[3 * a + 2])));
            }
            const int mbw = wave_max(__float_as_int(mb));
            int light_w = 0;
            if constexpr (!F32) {
                wmin = smallest_weight();
                light_w = (int)__popcll(__ballot(in_tile && wmin < LIGHT_W));
            }
            if (lane == 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    red_i[a][wv] = mn[a];
                    red_i[3 + a][wv] = mx[a];
                }
                red_i[6][wv] = mbw;
                red_i[7][wv] = light_w;
            }
            __syncthreads();
            if constexpr (FUSED) {  // every gather is done: clear the staged node box, keeping the tile zero
                for (int t = tid; t < 2 * ngs; t += NT) tq[t] = 0.0;
                __syncthreads();
            }
            int hi[3], mbk = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = INT_MAX;
                hi[a] = INT_MIN;
            }
#pragma unroll
            for (int k = 0; k < NT / 64; ++k) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    lo[a] = min(lo[a], red_i[a][k]);
                    hi[a] = max(hi[a], red_i[3 + a][k]);
                }
                mbk = max(mbk, red_i[6][k]);
                if constexpr (!F32) lights += __builtin_amdgcn_readfirstlane(red_i[7][k]);
            }
            // the chunk's momentum bound, above the rounding of the particles' own bounds and of m, and
            // its scale: every contribution w (m + K) <= 27/64 2 K < 2^em
            m_bound = 1.0001f * __int_as_float(mbk);
            (void)frexpf(F32 ? 0.421875f * __int_as_float(mbk) : 0.84375f * m_bound, &em);
            em = min(max(em, -70), 77);
            if (hi[0] >= lo[0]) {
#pragma unroll
                for (int a = 0; a < 3; ++a) ext[a] = hi[a] - lo[a] + 1;
                nt = ext[0] * ext[1] * ext[2];
                R = pitch_row(ext[0]);
                Q = pitch_plane(R, ext[1]);
            }
            // no room in the tile or in this workgroup's staging slice: the chunk goes to global atomics
            if (Q * ext[2] > CT || used + nt > slice) nt = -1;
            if (!ch.tile) nt = -1;  // a registration list was full at the rebuild
            if (nt < 0 && tid == 0) atomicAdd(&ctl64(ctl, blockIdx.x)[CTL64_FALLBACK_CHUNKS], 1ull);
            off = slice0 + used;
            if (nt > 0) {
                used += nt;
                // Lanes of one cell add to the same words, one after another: where the chunk holds 8
                // particles and more per cell of its box, the tile is kept in up to 16 copies that the
                // lanes take in turn.  (Water that ASFLIP has pressed into a corner holds thousands of
                // particles in one cell: 48.4 -> 23.8 us at 143K.  From 4 a cell on it would be 22.3
                // there, but 97.9 -> 105.3 for 1.39M snow particles, 8 to a cell, whose deal over the
                // lanes already keeps a cell's particles apart.)
                const int cells = (ext[0] - 2) * (ext[1] - 2) * (ext[2] - 2);
                if (8 * cells <= count)
                    while (copies < 16 && 4 * copies * cells <= count && 2 * copies * (Q * ext[2] | 1) <= CT) copies *= 2;
                copies = __builtin_amdgcn_readfirstlane(copies);
            }
            // (the tile is all zero here: cleared at the start, and every node a chunk touched is
            // zeroed again as it is stored)
            if (tid == 0)
                box[c] = nt > 0 ? make_int4(lo[0] | (lo[1] << 10) | (lo[2] << 20), ext[0] | (ext[1] << 8) | (ext[2] << 16),
                                            off, 0)
                                : make_int4(0, 0, 0, 0);
        }

        // ---- phase 2: scatter
        {
            const unsigned long long g = __ballot(have && ok && (GLOBAL_ONLY || !in_zone || nt <= 0));
            if (g && lane == 0)
                atomicAdd(&ctl64(ctl, blockIdx.x * (NT / 64) + wv)[CTL64_GLOBAL_PARTICLES], (unsigned long long)__popcll(g));
            // in-zone particles that lost the tile: a rebuild would shrink their chunk's box again
            const unsigned long long fb = __ballot(have && ok && !GLOBAL_ONLY && in_zone && nt <= 0);
            if (fb && lane == 0) atomicAdd(&ctl[CTL_FB + parity], (int)__popcll(fb));
        }
#if MPM_WEIGHTS_IN_LDS  // (a barrier separates the store from this load)
        if (have) {
#pragma unroll
            for (int k = 0; k < 9; ++k) st.w[k / 3][k % 3] = wpark[k * NT + tid];
        }
#endif
        const bool tiled = !GLOBAL_ONLY && have && ok && in_zone && nt > 0;
        int tb = 0;  // tile index of the stencil's first node
        if constexpr (F32) {
            const bool any_tiny = __any(tiled && smallest_weight() < TINY_W);
            if (tiled) {
                tb = (st.base[0] - lo[0]) + R * (st.base[1] - lo[1]) + Q * (st.base[2] - lo[2]) +
                     (copies > 1 ? (tid & (copies - 1)) * (Q * ext[2] | 1) : 0);
                unsigned long long* tu = reinterpret_cast<unsigned long long*>(tq);
                const float m_scale = ldexpf(1.0f, FRAC_M_F32 - em), m_unit = ldexpf(1.0f, em - FRAC_M_F32);
                float qs[3], As[9];  // in momentum units (exact: a power-of-two scale)
#pragma unroll
                for (int a = 0; a < 3; ++a) qs[a] = q[a] * m_scale;
#pragma unroll
                for (int k = 0; k < 9; ++k) As[k] = Ad[k] * m_scale;
                auto scatter = [&](auto check) {  // (the test of each term only in waves that need it)
                    constexpr bool CHECK = decltype(check)::value;
#pragma unroll
                    for (int o2 = 0; o2 < 3; ++o2)
#pragma unroll
                        for (int o1 = 0; o1 < 3; ++o1) {
                            const float wyz = st.w[1][o1] * st.w[2][o2];
                            float m0 = qs[0] + o1 * As[1] + o2 * As[2];
                            float m1 = qs[1] + o1 * As[4] + o2 * As[5];
                            float m2 = qs[2] + o1 * As[7] + o2 * As[8];
                            const int row = tb + R * o1 + Q * o2;
#pragma unroll
                            for (int o0 = 0; o0 < 3; ++o0) {
                                const float w = wyz * st.w[0][o0];
                                const int t = row + o0;
                                if (!CHECK || w >= TINY_W) {
                                    atomicAdd(&tu[t], fixed64(w * W_SCALE_F32));
                                    atomicAdd(&tu[CT + t], fixed64(w * m0));
                                    atomicAdd(&tu[2 * CT + t], fixed64(w * m1));
                                    atomicAdd(&tu[3 * CT + t], fixed64(w * m2));
                                } else {  // rare: to the node's global accumulator, in FP32
                                    const int gx = st.base[0] + o0, gy = st.base[1] + o1, gz = st.base[2] + o2;
                                    const int bk = (((gz >> 2) + 1) * NB + ((gy >> 2) + 1)) * NB + ((gx >> 2) + 1);
                                    float* a = acc + 4 * ((int64_t)(brick_base + bk) * BLOCK_NODES + (gx & 3) +
                                                          ((gy & 3) << 2) + ((gz & 3) << 4));
                                    unsafeAtomicAdd(a + 0, w * M.mp);
                                    unsafeAtomicAdd(a + 1, w * m0 * m_unit);
                                    unsafeAtomicAdd(a + 2, w * m1 * m_unit);
                                    unsafeAtomicAdd(a + 3, w * m2 * m_unit);
                                    acc_dirty[brick_base + bk] = 1;
                                }
                                m0 += As[0];
                                m1 += As[3];
                                m2 += As[6];
                            }
                        }
                };
                if (any_tiny)
                    scatter(std::true_type{});
                else
                    scatter(std::false_type{});
            }
        } else if (tiled) {
            tb = (st.base[0] - lo[0]) + R * (st.base[1] - lo[1]) + Q * (st.base[2] - lo[2]) +
                     (copies > 1 ? (tid & (copies - 1)) * (Q * ext[2] | 1) : 0);
            unsigned long long* tu = reinterpret_cast<unsigned long long*>(tq);
            // weights times DENORM_SPLIT (in the z weights), momentum with the rest of the scale
            double wx[3], wy[3], wz[3], ax[3], ay[3], az[3], mz[3];
            const float ms = ldexpf(1.0f, FRAC_M - 74 - em);  // 2^(FRAC_M - em - 1074) / DENORM_SPLIT
            const double k = (double)m_bound * (double)ms;
            const double mark = wmin <= 0x1p-54f ? 0x1p-1074 : 0.0;  // (one unit)
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                wx[o] = (double)st.w[0][o];
                wy[o] = (double)st.w[1][o];
                wz[o] = (double)st.w[2][o] * DENORM_SPLIT;
                mz[o] = (double)(q[o] * ms) + k;
                ax[o] = (double)(Ad[3 * o] * ms);
                ay[o] = (double)(Ad[3 * o + 1] * ms);
                az[o] = (double)(Ad[3 * o + 2] * ms);
            }
#pragma unroll
            for (int o2 = 0; o2 < 3; ++o2) {
                double my[3] = {mz[0], mz[1], mz[2]};
#pragma unroll
                for (int o1 = 0; o1 < 3; ++o1) {
                    const double wyz = wy[o1] * wz[o2];
                    double m[3] = {my[0], my[1], my[2]};
                    const int row = tb + R * o1 + Q * o2;
#pragma unroll
                    for (int o0 = 0; o0 < 3; ++o0) {
                        const double w = wyz * wx[o0];
                        const int t = row + o0;
                        atomicAdd(&tu[t], (unsigned long long)__double_as_longlong(fma(w, 0x1p-20, mark)));
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            atomicAdd(&tu[(a + 1) * CT + t], (unsigned long long)__double_as_longlong(w * m[a]));
                            m[a] += ax[a];
                        }
                    }
#pragma unroll
                    for (int a = 0; a < 3; ++a) my[a] += ay[a];
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) mz[a] += az[a];
            }
        }

        // ---- store the tile to the chunk's staging slot
        if (!GLOBAL_ONLY) {
            __syncthreads();
            if (copies > 1) {  // (whole-number sums: the same in any order)
                unsigned long long* tu = reinterpret_cast<unsigned long long*>(tq);
                const int nodes = Q * ext[2];
                for (int t = tid; t < nodes; t += NT)
#pragma unroll
                    for (int ch4 = 0; ch4 < 4; ++ch4) {
                        unsigned long long sum = tu[ch4 * CT + t];
                        for (int k = 1; k < copies; ++k) {
                            unsigned long long& w = tu[ch4 * CT + t + k * (nodes | 1)];
                            sum += w;
                            w = 0ull;
                        }
                        tu[ch4 * CT + t] = sum;
                    }
                __syncthreads();
            }
            float4* slot = stage + off;
            const int e01 = ext[0] * ext[1];
            const float r01 = 1.0f / (float)(e01 > 0 ? e01 : 1), r0 = 1.0f / (float)(ext[0] > 0 ? ext[0] : 1);
            const double m_unit = ldexp(1.0, em - FRAC_M), mass_unit = 0x1p-54 * (double)M.mp;
            const double k_unit = 0x1p-54 * (double)m_bound;
            const unsigned long long weak_sum = (unsigned long long)lights << WEAK_SHIFT;
            for (int u = tid; u < nt; u += NT) {  // staged in the tight box layout
                const int z = div_small(u, r01), u01 = u - z * e01;
                const int y = div_small(u01, r0), xx = u01 - y * ext[0];
                const int t = xx + R * y + Q * z;
                const unsigned long long* tu = reinterpret_cast<const unsigned long long*>(tq);
                const unsigned long long wsum = tu[t];
                if constexpr (F32) {
                    const double mu = (double)ldexpf(1.0f, em - FRAC_M_F32);
                    slot[u] = make_float4((float)((double)(long long)wsum * (0x1p-51 * (double)M.mp)),
                                          (float)((double)(long long)tu[CT + t] * mu),
                                          (float)((double)(long long)tu[2 * CT + t] * mu),
                                          (float)((double)(long long)tu[3 * CT + t] * mu));
                } else if (wsum == 0ull || wsum >= weak_sum) {
                    const double wd = (double)wsum, kw = k_unit * wd;  // K times the weight sum
                    slot[u] = make_float4((float)(wd * mass_unit), (float)((double)tu[CT + t] * m_unit - kw),
                                          (float)((double)tu[2 * CT + t] * m_unit - kw),
                                          (float)((double)tu[3 * CT + t] * m_unit - kw));
                } else {
                    weak[atomicAdd(&n_weak, 1)] = (unsigned short)(xx | (y << 5) | (z << 10));
                }
#pragma unroll
                for (int ch4 = 0; ch4 < 4; ++ch4) tq[ch4 * CT + t] = 0.0;  // ready for the next chunk
            }
            __syncthreads();
            const int nw = n_weak;  // uniform over the workgroup
            if (nw > 0) {
                // Only a particle with a weight below the weak nodes' bound can have added to one: a few
                // lanes of a wave.  The wave takes such particles one by one and tests 64 weak nodes at a
                // time, a lane each.
                const float bound = (float)lights * (0.5f * LIGHT_W);
                const unsigned long long tiny = __ballot(tiled && wmin < bound);
                for (int k0 = 0; tiny && k0 < nw; k0 += 64) {
                    const bool mine = k0 + lane < nw;
                    const int e = mine ? weak[k0 + lane] : 0, wx = e & 31, wy = (e >> 5) & 31, wz = e >> 10;
                    double* node = tq + wx + R * wy + Q * wz;
                    for (unsigned long long m = tiny; m; m &= m - 1) {
                        const int l = __builtin_ctzll(m);
                        auto get = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
                        const unsigned o0 = lo[0] + wx - __builtin_amdgcn_readlane(st.base[0], l);
                        const unsigned o1 = lo[1] + wy - __builtin_amdgcn_readlane(st.base[1], l);
                        const unsigned o2 = lo[2] + wz - __builtin_amdgcn_readlane(st.base[2], l);
                        const bool hit = mine && o0 <= 2u && o1 <= 2u && o2 <= 2u;
                        if (!__any(hit)) continue;
                        float w[3][3], am[9], qm[3];
#pragma unroll
                        for (int k = 0; k < 9; ++k) {
                            w[k / 3][k % 3] = get(st.w[k / 3][k % 3]);
                            am[k] = get(Ad[k]);
                        }
#pragma unroll
                        for (int a = 0; a < 3; ++a) qm[a] = get(q[a]);
                        if (hit) {
                            const double wt = (double)(pick3(w[1], o1) * pick3(w[2], o2)) * (double)pick3(w[0], o0);
                            unsafeAtomicAdd(node, wt);
#pragma unroll
                            for (int a = 0; a < 3; ++a)
                                unsafeAtomicAdd(node + (a + 1) * CT,
                                                wt * (double)(qm[a] + (float)o1 * am[3 * a + 1] + (float)o2 * am[3 * a + 2] +
                                                              (float)o0 * am[3 * a]));
                        }
                    }
                }
                __syncthreads();
                if (tid == 0) n_weak = 0;  // (every thread has read it)
                for (int k = tid; k < nw; k += NT) {
                    const int e = weak[k], wx = e & 31, wy = (e >> 5) & 31, wz = e >> 10;
                    double* node = tq + wx + R * wy + Q * wz;
                    slot[wx + ext[0] * (wy + ext[1] * wz)] =
                        make_float4((float)(node[0] * (double)M.mp), (float)node[CT], (float)node[2 * CT], (float)node[3 * CT]);
#pragma unroll
                    for (int ch4 = 0; ch4 < 4; ++ch4) node[ch4 * CT] = 0.0;
                }
                __syncthreads();
            }
        }

        // ---- particles without a tile: straight to the global accumulators
        if (have && ok && !tiled) {
            if (!in_zone)
                activate_blocks(st, NB, brick_base, brick_state, ovf, &ctl[CTL_OVF + parity], nbricks, err);
            int xo[3], yo[3], zo[3];
            axis_offsets(st.base[0], 1, 0, xo);
            axis_offsets(st.base[1], NB, 2, yo);
            axis_offsets(st.base[2], NB * NB, 4, zo);
            float* accs = acc + 4 * (int64_t)brick_base * BLOCK_NODES;
            {  // the stencil's nodes lie in blocks (base >> 2) + 1 and ((base + 2) >> 2) + 1 per axis
                int* dirty = acc_dirty + brick_base;
                const int bl[3] = {(st.base[0] >> 2) + 1, (st.base[1] >> 2) + 1, (st.base[2] >> 2) + 1};
                const int bh[3] = {((st.base[0] + 2) >> 2) + 1, ((st.base[1] + 2) >> 2) + 1,
                                   ((st.base[2] + 2) >> 2) + 1};
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    dirty[((k & 4 ? bh[2] : bl[2]) * NB + (k & 2 ? bh[1] : bl[1])) * NB + (k & 1 ? bh[0] : bl[0])] = 1;
            }
#pragma unroll
            for (int o2 = 0; o2 < 3; ++o2)
#pragma unroll
                for (int o1 = 0; o1 < 3; ++o1) {
                    const float wyz = st.w[1][o1] * st.w[2][o2];
                    float m0 = q[0] + o1 * Ad[1] + o2 * Ad[2];
                    float m1 = q[1] + o1 * Ad[4] + o2 * Ad[5];
                    float m2 = q[2] + o1 * Ad[7] + o2 * Ad[8];
#pragma unroll
                    for (int o0 = 0; o0 < 3; ++o0) {
                        const float w = wyz * st.w[0][o0];
                        float* a = accs + 4 * (xo[o0] + yo[o1] + zo[o2]);
                        unsafeAtomicAdd(a + 0, w * M.mp);
                        unsafeAtomicAdd(a + 1, w * m0);
                        unsafeAtomicAdd(a + 2, w * m1);
                        unsafeAtomicAdd(a + 3, w * m2);
                        m0 += Ad[0];
                        m1 += Ad[3];
                        m2 += Ad[6];
                    }
                }
        }
    }
    if constexpr (FUSED) {
        if (__ballot(left) != 0ull && (threadIdx.x & 63) == 0) {
            if (__hip_atomic_load(&ctl[CTL_REBUILD], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 &&
                atomicExch(&ctl[CTL_REBUILD], 1) == 0 && host_flag)
                __hip_atomic_store(host_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) ctl[CTL_STEP] += 1;  // the G2P part completed a substep
    }
    if (err) atomicOr(&ctl[CTL_ERROR], (int)err);
    if (SURM != 0 && (threadIdx.x & 63) == 0) {
        unsigned long long* c64 = ctl64(ctl, blockIdx.x * (NT / 64) + (threadIdx.x >> 6));
        if (n_sur) atomicAdd(&c64[CTL64_SUR_PARTICLES], (unsigned long long)n_sur);
        if (n_fb) atomicAdd(&c64[CTL64_SUR_FALLBACKS], (unsigned long long)n_fb);
    }
}


// Land the deferred deformation update of every particle with its scene's
// snow map -- exact, closed form (no SVD) or the network -- the way P2G
// applies it, for contexts where some snow scene takes a map without SVD.
// One chunk per workgroup pass (a chunk holds one scene, so the network runs
// on whole waves of one scene).
template <int SURM, int NT>
__global__ __launch_bounds__(NT) void k_materialize_map(float* __restrict__ S, int64_t cap,
                                                        const Chunk* __restrict__ chunks, const int* __restrict__ ctl,
                                                        Scenes T) {
    struct Empty {};
    __shared__ typename std::conditional<SURM == 2, mlp::NetLds16, Empty>::type net;
    __shared__ __attribute__((aligned(16))) float sur_stage[SURM == 2 ? NT / 64 * mlp::FWD_STAGE : 1];
    if constexpr (SURM == 2) {
        if (T.sur_theta) mlp::load_net16<NT>(net, T.sur_theta, T.sur_norm);
        __syncthreads();
    }
    const int nchunk = ctl[CTL_NCHUNK];
    const int tid = threadIdx.x, wv = tid >> 6;
    for (int c = blockIdx.x; c < nchunk; c += gridDim.x) {
        const Chunk ch = chunks[c];
        const Scene& sc = T.scene[ch.scene];
        const Mat M = sc.M;
        const bool have = tid < ch.count;
        const int p = ch.start + (have ? tid : 0);
        float C[9], F[9], s = 1.0f, tau[6];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            C[k] = have ? field(S, FC + k, p, cap) : 0.0f;
            F[k] = have ? field(S, FF + k, p, cap) : ((k % 4 == 0) ? 1.0f : 0.0f);
        }
        if (have) s = field(S, FS, p, cap);
        bool fb = false;
        if (sc.ret != 0 && M.kind == MPM_SNOW) {  // uniform over the workgroup
            if constexpr (SURM == 2) {
                if (sc.ret == 1)
                    snow_without_svd<true>(&net, sur_stage + wv * mlp::FWD_STAGE, T, sc, sc.P.dt, 1, have, C, F, s, tau, fb);
                else
                    snow_without_svd<false>(&net, sur_stage, T, sc, sc.P.dt, 1, have, C, F, s, tau, fb);
            } else {
                snow_without_svd<false>(nullptr, nullptr, T, sc, sc.P.dt, 1, have, C, F, s, tau, fb);
            }
        } else if (have) {
            material_step(M, sc.P.dt, 1, C, F, s, tau);
        }
        if (have) {
            if (M.kind != MPM_WATER) {
#pragma unroll
                for (int k = 0; k < 9; ++k) field(S, FF + k, p, cap) = F[k];
            }
            if (M.kind != MPM_JELLY) field(S, FS, p, cap) = s;
        }
    }
}

#define MPM_P2G_PARAMS                                                                                          \
    float *__restrict__ S, int64_t cap, const Chunk *__restrict__ chunks, int *__restrict__ ctl,               \
        float *__restrict__ acc, int *__restrict__ acc_dirty, float4 *__restrict__ stage, int stage_nodes,     \
        int4 *__restrict__ box,                                                                                 \
        int *__restrict__ brick_state, int *__restrict__ ovf, int parity, Scenes T, int pending, int nbricks, \
        int act, const float4 *__restrict__ vel, int *__restrict__ host_flag, int fb_limit
#define MPM_P2G_ARGS \
    S, cap, chunks, ctl, acc, acc_dirty, stage, stage_nodes, box, brick_state, ovf, parity, T, pending, nbricks, act, vel, \
        host_flag, fb_limit

template <bool GLOBAL_ONLY, int NT, int SURM>
__global__ __launch_bounds__(NT) void k_p2g(MPM_P2G_PARAMS) {
    p2g_body<GLOBAL_ONLY, NT, SURM, false>(MPM_P2G_ARGS);
}

template <int NT, int SURM>
__global__ __launch_bounds__(NT) void k_p2g_f32(MPM_P2G_PARAMS) {
    p2g_body<false, NT, SURM, false, true>(MPM_P2G_ARGS);
}

// The fused form holds the gathered v and C beside the P2G state; four
// waves per SIMD (at most 128 VGPRs) keep it as resident as the plain form.
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_p2g_fused(MPM_P2G_PARAMS) {
    p2g_body<false, NT, 0, true>(MPM_P2G_ARGS);
}

#undef MPM_P2G_PARAMS
#undef MPM_P2G_ARGS

}  // namespace

int p2g_grid_size(int cus, int chunk) {
    const int nt = chunk_threads(chunk);
    const void* fn = nt == 128   ? reinterpret_cast<const void*>(k_p2g<false, 128, 0>)
                     : nt == 256 ? reinterpret_cast<const void*>(k_p2g<false, 256, 0>)
                                 : reinterpret_cast<const void*>(k_p2g<false, 512, 0>);
    // Four times the resident workgroups (at most 4096 threads per CU): the
    // chunks of the block-sorted list differ in cost (fill, box size), and
    // with each workgroup taking every stride-th chunk of its XCD's slice,
    // more and shorter-lived workgroups even the load out (twice the
    // resident count: 146.6 us, four times: 140.9 us per launch on the
    // 1.28M-particle snow scene, frames 2-40).
    int occ = 4 * wgs_per_cu(fn, nt);
    if (occ > 4096 / nt) occ = 4096 / nt;
    const int g = cus * occ;
    return g < 8 ? 8 : (g / 8) * 8;
}

void enqueue_p2g(hipStream_t st, const Launch& L, const Scenes& T, float* S, int64_t cap, const Chunk* chunks,
                 int* ctl, GridBuffers& G, int* brick_state, int pending, int parity, int global_atomics,
                 int nbricks, int chunk, int act, int fused, int* host_flag, int fb_limit, int f32) {
    const int nt = chunk_threads(chunk);
    const int surm = T.sur_any;  // 0, 1 (closed form) or 2 (network)
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(L.p2g_grid), dim3(threads), 0, st, S, cap, chunks, ctl, G.acc, G.acc_dirty, G.stage,
                           G.stage_nodes, G.box, brick_state, G.ovf[parity], parity, T, pending, nbricks, act, G.vel,
                           host_flag, fb_limit);
    };
#define MPM_LAUNCH_P2G_NT(GO, SU)                                                              \
    do {                                                                                       \
        if (nt == 128) launch(k_p2g<GO, 128, SU>, 128);                                        \
        else if (nt == 256) launch(k_p2g<GO, 256, SU>, 256);                                   \
        else launch(k_p2g<GO, 512, SU>, 512);                                                  \
    } while (0)
#define MPM_LAUNCH_P2G_F32_NT(SU)                                                              \
    do {                                                                                       \
        if (nt == 128) launch(k_p2g_f32<128, SU>, 128);                                        \
        else if (nt == 256) launch(k_p2g_f32<256, SU>, 256);                                   \
        else launch(k_p2g_f32<512, SU>, 512);                                                  \
    } while (0)
    if (fused) {  // callers check: tile path, exact map
        if (nt == 128) launch(k_p2g_fused<128>, 128); else if (nt == 256) launch(k_p2g_fused<256>, 256); else launch(k_p2g_fused<512>, 512);
    } else if (f32 && !global_atomics) {
        if (surm == 2) MPM_LAUNCH_P2G_F32_NT(2); else if (surm == 1) MPM_LAUNCH_P2G_F32_NT(1); else MPM_LAUNCH_P2G_F32_NT(0);
    } else if (global_atomics) {
        if (surm == 2) MPM_LAUNCH_P2G_NT(true, 2); else if (surm == 1) MPM_LAUNCH_P2G_NT(true, 1); else MPM_LAUNCH_P2G_NT(true, 0);
    } else {
        if (surm == 2) MPM_LAUNCH_P2G_NT(false, 2); else if (surm == 1) MPM_LAUNCH_P2G_NT(false, 1); else MPM_LAUNCH_P2G_NT(false, 0);
    }
#undef MPM_LAUNCH_P2G_NT
#undef MPM_LAUNCH_P2G_F32_NT
}

void enqueue_materialize_map(hipStream_t st, const Launch& L, const Scenes& T, float* S, int64_t cap,
                             const Chunk* chunks, const int* ctl, int chunk) {
    const int nt = chunk_threads(chunk);
    const int grid = L.p2g_grid;
#define MPM_LAUNCH_MAT(SU)                                                                                        \
    do {                                                                                                          \
        if (nt == 128) hipLaunchKernelGGL((k_materialize_map<SU, 128>), dim3(grid), dim3(128), 0, st, S, cap, chunks, ctl, T); \
        else if (nt == 256) hipLaunchKernelGGL((k_materialize_map<SU, 256>), dim3(grid), dim3(256), 0, st, S, cap, chunks, ctl, T); \
        else hipLaunchKernelGGL((k_materialize_map<SU, 512>), dim3(grid), dim3(512), 0, st, S, cap, chunks, ctl, T); \
    } while (0)
    if (T.sur_any == 2) MPM_LAUNCH_MAT(2); else MPM_LAUNCH_MAT(1);
#undef MPM_LAUNCH_MAT
}

}  // namespace mpm

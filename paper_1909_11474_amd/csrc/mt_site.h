// Per-atom evaluation of the Tersoff site energy for one candidate: the
// minimal potential, or the nine-parameter Tersoff form.
//
// One thread owns one atom i with M bonds (compile-time M, padded bonds have
// f_C = f_C' = 0 and contribute nothing).  For a candidate parameter record it
// computes the site energy U_i and the bond gradients G_ij = dU_i/dr_ij:
//
//   zeta_ij = beta sum_{k != j} f_C(r_ik) (cos theta_ijk - h)^2          (Sec. II.A Eq. 7, Sec. II.B Eq. 10)
//   b_ij = (1 + zeta^n)^(-1/(2n)) (b = 1 at zeta = 0)                    (Sec. II.A Eq. 6)
//   U_i = 1/2 sum_j f_C(r_ij) [f_R - b_ij f_A]                            (Sec. II.A Eqs. 2-3)
//   with S = 2:  f_R = D0 x^2,  f_A = 2 D0 x,  x = exp(-alpha (r - r0))  (Sec. II.B Eqs. 11-14)
//
// G_ij is the exact derivative of U_i.  Writing C_j = -f_C fA b'/2 for the
// coefficient of d zeta_ij, c~_j = 2 beta C_j, t_jk = cos_jk - h and
// q_jk = (c~_j f_C,k + c~_k f_C,j) t_jk, the gradient decomposes into a radial
// part along r^_j and a transverse sum:
//   G_j = [ D_j + f_C'_j/2 sum_k c~_k t_jk^2 - (1/r_j) r^_j . V_j ] r^_j + (1/r_j) V_j,
//   V_j = sum_k q_jk r^_k,
//   D_j = 1/2 [ f_C'_j (f_R - b f_A) + f_C,j alpha (b f_A - 2 f_R) ]
// (the radial term uses sum_k q_jk cos_jk = r^_j . V_j).  Every unordered bond
// pair (j, k) is visited once in each of the forward (zeta) and backward
// (gradient) sweeps; the float minimal potential above kPairMax neighbours takes
// both from moments over the bonds instead.
//
// The Tersoff form (Sec. II.A Eqs. 2-8 with Eqs. 11-14 for general S) replaces
// beta (cos - h)^2 by g^T(theta), t^2 by g^T in the P sums, t by g^T'/2 in q_jk,
// and takes f_R, f_A with their own exponents lambda = alpha sqrt(2S),
// mu = alpha sqrt(2/S); then D_j = 1/2 [f_C' (f_R - b f_A) + f_C (mu b f_A - lambda f_R)].
//
// S is the arithmetic type (float or double); the code is written once for both.
#pragma once

#include <type_traits>

#include "mt_common.h"

namespace mt {

// Mom: the geometry serves many candidates (batched fitness and gradient), so the
// float minimal form takes moments above kPairMax neighbours.  The evaluation and
// two-pass kernels run one or a few candidates a block and are bound by latency:
// the moments' registers (3 M + 9 more) spill there and cost more than the pair sums.
// Evaluations in float, 500 close-packed atoms 26.0 us with pairs, 30.0 with moments;
// six cells of 14 neighbours x 64 candidates 42 and 51 us; fitness of a 1,500-atom
// packing x 400 138 and 146 us.
template <typename S, int M, bool Full = false, bool Mom = true>
struct Geo {
    static constexpr int NP = M * (M - 1) / 2;
    static constexpr bool kCache = NP <= 15;       // keep cos(theta) in registers for M <= 6
    static constexpr bool kMoments = Mom && !Full && sizeof(S) == 4 && M > kPairMax;
    S ux[M > 0 ? M : 1], uy[M > 0 ? M : 1], uz[M > 0 ? M : 1];
    double r[M > 0 ? M : 1];                      // float64 also in the float geometry: r - r0
    S rinv[M > 0 ? M : 1];
    S fc[M > 0 ? M : 1], hfcp[M > 0 ? M : 1];     // f_C and f_C'/2
    S cs[kCache && NP > 0 ? NP : 1];
    // The minimal form's angular function is (cos - h)^2, so bond j's sum over
    // the other bonds is a quadratic in h that no parameter enters:
    //   sum_k f_C (cos_jk - h)^2 = V + S (H - h)^2,
    // S = sum f_C, H = sum f_C cos / S, V = sum f_C (cos - H)^2, from the set's
    // table (float64 sums rounded once).  Both terms are positive, so nothing
    // cancels.
    S ss[kMoments ? M : 1], sh[kMoments ? M : 1], sv[kMoments ? M : 1];
    // sum f_C u u^T and sum f_C u over the bonds
    S txx, tyy, tzz, tyz, tzx, txy, mx, my, mz;

    __device__ __forceinline__ void load_moments(const SetDev& d, int atom, int rows) {
        if constexpr (kMoments) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const float4 a = m < rows ? d.gam[(size_t)m * d.N + atom] : make_float4(0.f, 0.f, 0.f, 0.f);
                ss[m] = a.x; sh[m] = a.y; sv[m] = a.z;
                rows_apart();
            }
            txx = tyy = tzz = tyz = tzx = txy = mx = my = mz = S(0);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const S fx = fc[m] * ux[m], fy = fc[m] * uy[m], fz = fc[m] * uz[m];
                mx += fx; my += fy; mz += fz;
                txx += fx * ux[m]; tyy += fy * uy[m]; tzz += fz * uz[m];
                tyz += fy * uz[m]; tzx += fz * ux[m]; txy += fx * uy[m];
            }
        }
    }

    // Loads stay in the order of the rows in the variants that fill the registers:
    // brought together, they spill values that the candidate loop then reloads
    // (without Mom the Tersoff form is faster as the compiler orders them: 500
    // close-packed atoms x 64 candidates in float 37 us, 40 in the rows' order; in
    // float64 its gradient is not, at four neighbours either: 64 candidates x 100 cells 86
    // us in the rows' order, 87).
    static __device__ __forceinline__ void rows_apart() {
        if constexpr (M > 6 ? Mom || !Full : sizeof(S) == 8 && Full && Mom) __builtin_amdgcn_sched_barrier(0);
    }

    __device__ __forceinline__ S length(int m) const { return (S)r[m]; }

    __device__ __forceinline__ S cosjk(int j, int k, int pidx) const {
        if constexpr (kCache && NP > 0) {
            return cs[pidx];
        } else {
            (void)pidx;
            return ux[j] * ux[k] + uy[j] * uy[k] + uz[j] * uz[k];
        }
    }

    // The cached angle cosines of the float geometry come from the set's pair
    // table, formed from the float64 unit vectors and rounded once; from float
    // unit vectors they carry up to ~2e-7 absolute error, which zeta passes on
    // to the energy through (cos - h)^2.
    // rows: neighbour rows the arrays hold (a variant wider than the set's
    // capacity reads the rows past it as padding bonds).  Lanes outside the
    // structure (not active) read the atom that they are given, with f_C = 0 on
    // every bond, so that they add nothing.  They take no branch of their own: at
    // its end the compiler may spill registers while those lanes are still off, and
    // a kernel of many spills then went on with whatever the spill slot held.
    __device__ __forceinline__ void load(const SetDev& d, int atom, bool active, int rows = M) {
        const int N = d.N;
        if constexpr (sizeof(S) == 4) {
            float rhi[M > 0 ? M : 1], rlo[M > 0 ? M : 1];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const size_t o = (size_t)m * N + atom;
                const bool ok = m < rows;
                const float4 a = ok ? d.gf.pk0[o] : make_float4(0.f, 0.f, 0.f, 3.f);
                const float4 b = ok ? d.gf.pk1[o] : make_float4(0.f, 0.f, 0.f, 0.f);
                ux[m] = a.x; uy[m] = a.y; uz[m] = a.z; rhi[m] = a.w; rlo[m] = b.x;
                rinv[m] = b.y; fc[m] = b.z; hfcp[m] = b.w;
                rows_apart();
            }
#pragma unroll
            for (int m = 0; m < M; ++m) r[m] = (double)rhi[m] + (double)rlo[m];
            if constexpr (kCache && NP > 0) {
                static_assert(M <= 6, "the pair table holds bonds 0-5");
                int p = 0;
#pragma unroll
                for (int j = 0; j < M; ++j)
#pragma unroll
                    for (int k = j + 1; k < M; ++k)
                        cs[p++] = k < rows ? d.gcs[(size_t)(k * (k - 1) / 2 + j) * N + atom] : S(0);
            }
        } else {
            const GeomArrays<double>& G = d.gd;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const size_t o = (size_t)m * N + atom;
                const bool ok = m < rows;
                ux[m] = ok ? G.ux[o] : S(0);
                uy[m] = ok ? G.uy[o] : S(0);
                uz[m] = ok ? G.uz[o] : S(0);
                r[m] = ok ? G.rhi[o] : S(3);
                rinv[m] = ok ? G.rinv[o] : S(0);
                fc[m] = ok ? G.fc[o] : S(0);
                hfcp[m] = ok ? G.hfcp[o] : S(0);
                rows_apart();
            }
            cache_cos();
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
            fc[m] = active ? fc[m] : S(0);
            hfcp[m] = active ? hfcp[m] : S(0);
        }
        load_moments(d, atom, rows);
    }

    __device__ __forceinline__ void cache_cos() {
        if constexpr (kCache && NP > 0) {
            int p = 0;
#pragma unroll
            for (int j = 0; j < M; ++j)
#pragma unroll
                for (int k = j + 1; k < M; ++k) cs[p++] = ux[j] * ux[k] + uy[j] * uy[k] + uz[j] * uz[k];
        }
    }
};

// Decoded parameters of one candidate.  Full selects the Tersoff angular
// function g^T and independent pair exponents (the nine-parameter form); the
// minimal potential has g = (cos - h)^2 and lambda = 2 mu.
template <typename S, bool Full = false>
struct Cand {
    static constexpr bool kFull = Full;
    S aA, aR, DR, DA, hmu, hlambda, zs, ccs, n, ninv2n, h;
    S gam, K, d2, Kd2;               // g^T = gam + K t^2 / (d2 + t^2)
    S valid;
    S hlo;                           // h - float(h): zeta of the float path
    double r0, aA64, aR64, DR64, DA64, ninv2n64;   // float64 energy terms
};

// Type of the site energy: float64 for the float path (its energy terms are
// evaluated in float64), the arithmetic type otherwise.
template <typename S>
struct EnergyOf { using type = S; };
template <>
struct EnergyOf<float> { using type = double; };

// The minimal record leaves the Tersoff form's fields unwritten; its candidate
// takes lambda = 2 mu, DA = 2 DR and does not read them.
template <typename S, bool Full>
__device__ __forceinline__ void load_cand(const Rec<S>& p, Cand<S, Full>& c) {
    c.aA = p.aA; c.DR = p.DR; c.DA = p.DA; c.hmu = p.hmu;
    c.zs = p.zs; c.ccs = p.ccs; c.n = p.n; c.ninv2n = p.ninv2n; c.h = p.h; c.hlo = p.hlo;
    c.valid = p.valid;
    c.r0 = p.r0; c.aA64 = p.aA64; c.DR64 = p.DR64; c.ninv2n64 = p.ninv2n64;
    if constexpr (Full) {
        c.aR = p.aR; c.hlambda = p.hlambda; c.aR64 = p.aR64; c.DA64 = p.DA64;
        c.gam = p.gam; c.K = p.K; c.d2 = p.d2; c.Kd2 = p.Kd2;
    } else {
        c.aR = S(2) * c.aA; c.hlambda = S(2) * c.hmu; c.aR64 = 2.0 * c.aA64; c.DA64 = 2.0 * c.DR64;
        c.gam = S(0); c.K = S(0); c.d2 = S(1); c.Kd2 = S(0);
    }
}

// Angular function and half its derivative for t = cos(theta) - h:
// minimal g = t^2, g'/2 = t; Tersoff g^T = gam + K t^2 / (d^2 + t^2),
// g'/2 = K d^2 t / (d^2 + t^2)^2 (Sec. II.A Eq. 8, written without the
// cancellation of 1 + c^2/d^2 - c^2/(d^2 + t^2)).
template <bool Full, typename S, typename P>
__device__ __forceinline__ S ang_g(const P& p, S t) {
    const S t2 = t * t;
    if constexpr (Full) return p.gam + (p.K * t2) * drcp(p.d2 + t2);
    else return t2;
}
template <bool Full, typename S, typename P>
__device__ __forceinline__ void ang_g_dg(const P& p, S t, S& gv, S& hg) {
    const S t2 = t * t;
    if constexpr (Full) {
        const S r = drcp(p.d2 + t2);
        gv = p.gam + (p.K * t2) * r;
        hg = ((p.Kd2 * t) * r) * r;
    } else {
        gv = t2;
        hg = t;
    }
}

// Make the compiler treat the values as changed here (no instruction is
// emitted): expressions of them after this point are recomputed, not reused.
template <typename T, int N>
__device__ __forceinline__ void opaque(T (&a)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(a[i]));
}

// Largest coordination whose backward sweep runs over unordered bond pairs
// (where it does not take moments).  Above it one bond at a time: more pair
// arithmetic, but four running sums instead of 4 M.  Float Tersoff form, 200
// candidates x 22 packings: 134 us at 6, 142 at 8, 153 at 10, 181 at 12.
template <typename S, bool Full, bool Mom = true>
constexpr int kPairwiseMax = Mom && Full && sizeof(S) == 4 ? 6 : 8;

// The site routine.  It hands each bond gradient G_j to sink(j, Gx, Gy, Gz);
// PerBond selects the one-bond-at-a-time backward sweep (for large M without
// moments), which emits G_j as soon as it is complete.
// SerialE64: keep the float64 energy chains of the bonds one after another
// (fewer live registers; a kernel with other wavefronts to switch to loses
// nothing), or let them interleave (a kernel that runs about one wavefront per
// SIMD needs the instruction-level parallelism).
// park: where the moment path leaves two values per bond between its sweeps
// (registers, or the bond's exchange slot).
template <typename S, int M>
struct ParkRegs {
    S a[M > 0 ? M : 1], b[M > 0 ? M : 1];
    __device__ __forceinline__ void put(int j, S x, S y) { a[j] = x; b[j] = y; }
    __device__ __forceinline__ void get(int j, S& x, S& y) const { x = a[j]; y = b[j]; }
};

template <typename S, int M, bool Energy64, bool PerBond, bool Full = false, bool SerialE64 = true, bool Mom = true,
          typename Sink, typename Park>
__device__ __forceinline__ void site_eval_sink(Geo<S, M, Full, Mom>& g, const Cand<S, Full>& p,
                                               typename EnergyOf<S>::type& U, Sink&& sink, Park&& park) {
    constexpr int MM = M > 0 ? M : 1;
    if constexpr (!Geo<S, M, Full, Mom>::kCache && M > 1) {
        // cos(theta) is not cached for larger M: keep the compiler from
        // hoisting the M (M - 1) / 2 values out of the candidate loop (they
        // would not fit in registers and go to scratch)
        opaque(g.ux);
        opaque(g.uy);
        opaque(g.uz);
    }
    // Energy64 (float path): the pair terms and the bond order of the energy
    // are evaluated with float64 exponentials (below), and zeta takes h as a
    // float hi/lo pair, so that a float rounding of h does not shift every
    // (cos - h)^2 of a candidate the same way.
    constexpr bool kE64 = Energy64 && std::is_same<S, float>::value;
    // the float copies of r and float64 copies of f_C are made per candidate:
    // hoisted out of the candidate loop they would hold 3 M registers
    if constexpr (kE64 && M > 0) {
        opaque(g.r);
        opaque(g.fc);
    }
    // Energy64: in float32 the rounding of f_R and b f_A (up to ~15 eV each
    // for parameters inside the fitting box) and the one-ulp errors of the
    // hardware exponentials reach 1e-6 eV per bond.  The exponentials whose
    // errors reach the energy at full weight, e^{-mu (r - r0)} and b, are
    // taken in float64 (the argument of b from the float logarithm of
    // 1 + zeta^n, whose error enters b damped by zeta^n / (1 + zeta^n) / 2n),
    // and the pair energy is formed in float64.  Their float32 roundings feed
    // the gradient.
    S usum = S(0);
    double usum64 = 0.0;
    // bond j's energy terms from its angular sum: c~_j and D_j of its gradient
    auto bond = [&](int j, S zeta, S& ccj, S& Dj) __attribute__((always_inline)) {
        const S z = zeta * p.zs;
        // zeta = 0 (no other neighbour inside the cutoff, or all at g = 0):
        // zeta^n = 0 exactly, so b = 1 and db/dzeta * zeta^n-terms vanish
        S zsafe, eA, zn, b;
        [[maybe_unused]] S eR;
        if constexpr (kE64) {
            const double dl = g.r[j] - p.r0;
            const double eA64 = exp2_acc(-(p.aA64 * dl));
            // log2 0 = -inf and 2^-inf = 0; the divisor below stays positive, and
            // is zeta itself down to the smallest normal value
            zn = dexp2(p.n * dlog2(z));
            zsafe = __builtin_fmaxf(z, 1.17549435e-38f);
            const double b64 = exp2_acc(p.ninv2n64 * (double)dlog2(1.f + zn));
            if constexpr (Full) {
                const double eR64 = exp2_acc(-(p.aR64 * dl));
                usum64 += (double)g.fc[j] * (p.DR64 * eR64 - b64 * (p.DA64 * eA64));
                eR = (float)eR64;
            } else {
                // DA = 2 DR, e_R = e_A^2
                usum64 += (double)g.fc[j] * (p.DR64 * eA64 * (eA64 - 2.0 * b64));
            }
            eA = (float)eA64;
            b = (float)b64;
        } else {
            const bool pos = z > S(0);
            zsafe = pos ? z : S(1);
            const S delta = (S)(g.r[j] - p.r0);
            eA = dexp2(-(p.aA * delta));
            if constexpr (Full) eR = dexp2(-(p.aR * delta));
            // formed before the selection: a branch around it splits the chain
            const S zne = dexp2(p.n * dlog2<true>(zsafe));
            zn = pos ? zne : S(0);
            b = dexp2(p.ninv2n * dlog2<true>(S(1) + zn));
        }
        const S onep = S(1) + zn;
        S fR;
        if constexpr (Full) fR = p.DR * eR;
        else fR = p.DR * (eA * eA);               // e_R = e_A^2
        const S fA = p.DA * eA;
        const S diff = fR - b * fA;           // one rounding (fused multiply-add)
        const S bfA = b * fA;
        if constexpr (!kE64) usum = usum + g.fc[j] * diff;
        // D = 1/2 [f_C' (f_R - b f_A) + f_C (mu b f_A - lambda f_R)]
        if constexpr (Full) Dj = g.hfcp[j] * diff + g.fc[j] * (p.hmu * bfA - p.hlambda * fR);
        else Dj = g.hfcp[j] * diff + (p.hmu * g.fc[j]) * (bfA - S(2) * fR);
        // c~ = -ZS f_C f_A db/dzeta with db/dzeta = -b zeta^n / (2 zeta (1 + zeta^n))
        ccj = (p.ccs * g.fc[j]) * (bfA * zn) * drcp_inf(zsafe * onep);
        // keep the scheduler from interleaving all M bonds' chains (about ten
        // live values each; float64 ones in the energy mode)
        if constexpr (PerBond || Geo<S, M, Full, Mom>::kMoments || (kE64 && SerialE64)) __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (Geo<S, M, Full, Mom>::kMoments) {
        // The pair sums of every bond from the moments over all bonds:
        //   sum_k (c~_j f_C,k + c~_k f_C,j) t_jk u_k = c~_j (T u_j - h m) + f_C,j (T~ u_j - h m~),
        //   sum_k c~_k t_jk^2 = u_j . T~ u_j - 2 h u_j . m~ + h^2 s~,
        // T = sum f_C u u^T, m = sum f_C u (no parameter in them) and T~, m~, s~
        // the same with c~ for f_C.  The bond's own term is radial in the first
        // (removed with the rest of V's radial part) and c~_j (1 - h)^2 in the
        // second.  About 55 operations per bond, where a sweep over ordered pairs
        // takes 12 per pair: bound by VALU issue either way (1,870 instructions a
        // step at M = 12), the M <= 12 launch of 500 candidates x 101 packings
        // takes 784 us against 969 us.
        S txx = S(0), tyy = txx, tzz = txx, tyz = txx, tzx = txx, txy = txx, mx = txx, my = txx, mz = txx,
          sc = txx;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            S t, c, Dj;
            if constexpr (kE64) t = (g.sh[j] - p.h) - p.hlo;
            else t = g.sh[j] - p.h;
            bond(j, g.sv[j] + (g.ss[j] * t) * t, c, Dj);
            park.put(j, c, Dj);
            const S cx = c * g.ux[j], cy = c * g.uy[j], cz = c * g.uz[j];
            sc += c;
            mx += cx; my += cy; mz += cz;
            txx += cx * g.ux[j]; tyy += cy * g.uy[j]; tzz += cz * g.uz[j];
            tyz += cy * g.uz[j]; tzx += cz * g.ux[j]; txy += cx * g.uy[j];
        }
        if constexpr (kE64) U = 0.5 * usum64; else U = S(0.5) * usum;
        mx *= p.h; my *= p.h; mz *= p.h;
        const S hx = p.h * g.mx, hy = p.h * g.my, hz = p.h * g.mz;
        const S h2s = (p.h * p.h) * sc, omh2 = (S(1) - p.h) * (S(1) - p.h);
#pragma unroll
        for (int j = 0; j < M; ++j) {
            S c, Dj;
            park.get(j, c, Dj);
            const S ux = g.ux[j], uy = g.uy[j], uz = g.uz[j], f = g.fc[j];
            const S yx = (txx * ux + txy * uy + tzx * uz) - mx;
            const S yy = (txy * ux + tyy * uy + tyz * uz) - my;
            const S yz = (tzx * ux + tyz * uy + tzz * uz) - mz;
            const S wx = (g.txx * ux + g.txy * uy + g.tzx * uz) - hx;
            const S wy = (g.txy * ux + g.tyy * uy + g.tyz * uz) - hy;
            const S wz = (g.tzx * ux + g.tyz * uy + g.tzz * uz) - hz;
            const S vx = f * yx + c * wx, vy = f * yy + c * wy, vz = f * yz + c * wz;
            const S pp = ((ux * yx + uy * yy + uz * yz) - (ux * mx + uy * my + uz * mz)) + (h2s - c * omh2);
            const S uv = ux * vx + uy * vy + uz * vz;
            const S rad = Dj + g.hfcp[j] * pp - uv * g.rinv[j];
            sink(j, rad * ux + vx * g.rinv[j], rad * uy + vy * g.rinv[j], rad * uz + vz * g.rinv[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    S zeta[MM], cc[MM], D[MM];
#pragma unroll
    for (int j = 0; j < M; ++j) zeta[j] = S(0);
    {
        int pidx = 0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
#pragma unroll
            for (int k = j + 1; k < M; ++k) {
                const S c = g.cosjk(j, k, pidx++);
                S t;
                if constexpr (kE64) t = (c - p.h) - p.hlo;
                else t = c - p.h;
                const S gv = ang_g<Full>(p, t);
                zeta[j] = zeta[j] + g.fc[k] * gv;
                zeta[k] = zeta[k] + g.fc[j] * gv;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < M; ++j) bond(j, zeta[j], cc[j], D[j]);
    if constexpr (kE64) U = 0.5 * usum64; else U = S(0.5) * usum;
    if constexpr (PerBond) {
        // One bond at a time, visiting each pair from both ends.
        // About 1.5x the backward arithmetic of the pairwise sweep below, but
        // only four running sums are live instead of 4 M, which keeps the
        // kernel out of scratch spills.  The barrier stops the compiler from
        // keeping the forward sweep's per-pair terms (about 2 M^2 values)
        // alive for reuse here.
        opaque(g.ux);
        opaque(g.uy);
        opaque(g.uz);
#pragma unroll
        for (int j = 0; j < M; ++j) {
            S vx = S(0), vy = vx, vz = vx, pp = vx;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                if (k == j) continue;
                const S c = g.ux[j] * g.ux[k] + g.uy[j] * g.uy[k] + g.uz[j] * g.uz[k];
                const S t = c - p.h;
                S gv, hg;
                ang_g_dg<Full>(p, t, gv, hg);
                const S q = (cc[j] * g.fc[k] + cc[k] * g.fc[j]) * hg;
                vx = vx + q * g.ux[k]; vy = vy + q * g.uy[k]; vz = vz + q * g.uz[k];
                if constexpr (Full) pp = pp + cc[k] * gv;
                else pp = pp + (cc[k] * t) * t;
            }
            const S uv = g.ux[j] * vx + g.uy[j] * vy + g.uz[j] * vz;
            const S rad = D[j] + g.hfcp[j] * pp - uv * g.rinv[j];
            sink(j, rad * g.ux[j] + vx * g.rinv[j], rad * g.uy[j] + vy * g.rinv[j],
                 rad * g.uz[j] + vz * g.rinv[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    S Vx[MM], Vy[MM], Vz[MM], Pp[MM];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        Vx[j] = Vy[j] = Vz[j] = Pp[j] = S(0);
    }
    {
        int pidx = 0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
#pragma unroll
            for (int k = j + 1; k < M; ++k) {
                const S c = g.cosjk(j, k, pidx++);
                const S t = c - p.h;
                S gv, hg;
                ang_g_dg<Full>(p, t, gv, hg);
                const S q = (cc[j] * g.fc[k] + cc[k] * g.fc[j]) * hg;
                Vx[j] = Vx[j] + q * g.ux[k]; Vy[j] = Vy[j] + q * g.uy[k]; Vz[j] = Vz[j] + q * g.uz[k];
                Vx[k] = Vx[k] + q * g.ux[j]; Vy[k] = Vy[k] + q * g.uy[j]; Vz[k] = Vz[k] + q * g.uz[j];
                Pp[j] = Pp[j] + cc[k] * gv;
                Pp[k] = Pp[k] + cc[j] * gv;
            }
        }
    }
    // sum_k q_jk cos_jk = u_j . V_j, so the radial part needs no per-pair term
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const S uv = g.ux[j] * Vx[j] + g.uy[j] * Vy[j] + g.uz[j] * Vz[j];
        const S rad = D[j] + g.hfcp[j] * Pp[j] - uv * g.rinv[j];
        sink(j, rad * g.ux[j] + Vx[j] * g.rinv[j], rad * g.uy[j] + Vy[j] * g.rinv[j],
             rad * g.uz[j] + Vz[j] * g.rinv[j]);
    }
}

// The site routine with the bond gradients returned in arrays.
template <typename S, int M, bool Energy64 = false, bool Full = false, bool SerialE64 = true, bool Mom = true>
__device__ __forceinline__ void site_eval(Geo<S, M, Full, Mom>& g, const Cand<S, Full>& p,
                                          typename EnergyOf<S>::type& U,
                                          S* __restrict__ Gx, S* __restrict__ Gy,
                                          S* __restrict__ Gz) {
    site_eval_sink<S, M, Energy64, (M > kPairwiseMax<S, Full, Mom>), Full, SerialE64, Mom>(
        g, p, U, [&](int j, S x, S y, S z) {
            Gx[j] = x;
            Gy[j] = y;
            Gz[j] = z;
        },
        ParkRegs<S, M>{});
}

// Cross-lane exchanges of a double, 32 bits at a time.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane l <-> 7 - l within 8 (opposite bit 2)
constexpr int kDppMirror = 0x140;      // lane l <-> 15 - l within 16 (opposite bit 3)

// Transpose step over lane bit m: lanes with the bit clear keep a (and add the
// partner's a), lanes with it set keep b.  permlane{16,32}_swap exchange the
// upper half of the first operand with the lower half of the second, so the
// two returned halves always sum to own kept value + partner's kept value.
template <int M>
__device__ __forceinline__ double tstep(double a, double b) {
    if constexpr (M == 32 || M == 16) {
        const long long ia = __double_as_longlong(a), ib = __double_as_longlong(b);
        const unsigned alo = (unsigned)ia, ahi = (unsigned)(ia >> 32);
        const unsigned blo = (unsigned)ib, bhi = (unsigned)(ib >> 32);
        unsigned r0lo, r1lo, r0hi, r1hi;
        if constexpr (M == 32) {
            auto l = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
            auto h = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
            r0lo = l[0]; r1lo = l[1]; r0hi = h[0]; r1hi = h[1];
        } else {
            auto l = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
            auto h = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
            r0lo = l[0]; r1lo = l[1]; r0hi = h[0]; r1hi = h[1];
        }
        const double x0 = __longlong_as_double(((long long)r0hi << 32) | r0lo);
        const double x1 = __longlong_as_double(((long long)r1hi << 32) | r1lo);
        return x0 + x1;
    } else {
        const bool h = (threadIdx.x & M) != 0;
        const double send = h ? a : b;
        const double keep = h ? b : a;
        constexpr int ctrl = M == 8 ? kDppMirror : (M == 4 ? kDppHalfMirror : (M == 2 ? kDppXor2 : kDppXor1));
        return keep + dpp_mov<ctrl>(send);
    }
}

template <int M>
__device__ __forceinline__ double bstep(double v) {
    constexpr int ctrl = M == 4 ? kDppHalfMirror : (M == 2 ? kDppXor2 : kDppXor1);
    return v + dpp_mov<ctrl>(v);
}

// Segmented transpose-reduction of 8 doubles over aligned groups of G lanes
// (G in 8, 16, 32, 64): three transpose steps over the top lane bits of the
// group, then butterfly steps over the rest.  Afterwards every lane holds the
// group sum of value index *vidx (bits of the transpose steps); lanes with
// (lane & (G/8 - 1)) == 0 are the writers.
template <int G>
__device__ __forceinline__ double group_reduce8_t(double* v, int* vidx) {
    constexpr int m1 = G / 2, m2 = G / 4, m3 = G / 8;
    const int lane = threadIdx.x & 63;
    double a4[4], a2[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) a4[k] = tstep<m1>(v[k], v[k + 4]);
#pragma unroll
    for (int k = 0; k < 2; ++k) a2[k] = tstep<m2>(a4[k], a4[k + 2]);
    double r = tstep<m3>(a2[0], a2[1]);
    if constexpr (m3 > 4) r = bstep<4>(r);
    if constexpr (m3 > 2) r = bstep<2>(r);
    if constexpr (m3 > 1) r = bstep<1>(r);
    *vidx = ((lane & m1) ? 4 : 0) + ((lane & m2) ? 2 : 0) + ((lane & m3) ? 1 : 0);
    return r;
}

__device__ __forceinline__ double group_reduce8(double* v, int g, int* vidx) {
    switch (g) {
        case 8: return group_reduce8_t<8>(v, vidx);
        case 16: return group_reduce8_t<16>(v, vidx);
        case 32: return group_reduce8_t<32>(v, vidx);
        default: return group_reduce8_t<64>(v, vidx);
    }
}

}  // namespace mt

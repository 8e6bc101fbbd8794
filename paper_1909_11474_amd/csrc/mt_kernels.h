// Device code of the evaluation kernels, shared by the per-family translation
// units (each instantiates the kernels of one precision / mode).
//
// Batched kernel.  A work item is (structure s, candidates c0 .. c0+nc-1).  A
// block of B threads holds R = B / npad_s replicas of the structure (npad_s is
// the atom count rounded up to 8/16/32/64 or to a multiple of 64), one atom per
// thread, or fewer where its LDS does not hold as many exchanges (the last
// wavefronts are idle then); replica q evaluates candidates c0 + q, c0 + q + R,
// ...  At the start of an item the block decodes the item's parameter sets into
// LDS; the bond geometry of the thread's atom is loaded once into registers and
// reused for every candidate.  Forces need the other atom's bond gradient
// (F_i = sum_j G_ij - G_ji): every thread writes its bond gradients to its
// exchange slots in LDS and reads back the reverse bonds.  A replica of up to
// 64 atoms lives inside one wavefront, whose LDS accesses are ordered, so it
// needs no barrier; larger replicas synchronise the block.  Per-atom energy,
// virial and squared force residual are reduced in float64 over aligned lane
// groups (transpose reduction over DPP / permlane exchanges), the wavefronts of
// a larger replica in LDS after that, and written to one partial-sum slot per
// (candidate, structure); the finalize kernels add the slots in a fixed order,
// so results are deterministic.
//
// Coordination classes.  Atoms inside a structure are sorted by coordination
// and each wavefront runs the variant compiled for its largest coordination M,
// so control flow is uniform.  A kernel instance serves one class MC: it holds
// the variants M = LO..MC (a wavefront with M < LO runs the LO variant with
// padded bonds), and a structure is routed to the smallest class that covers
// its largest coordination.  Register allocation then follows the class, so
// diamond-like structures (M <= 4) run at high occupancy.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "mt_host.h"
#include "mt_site.h"

namespace mt {

// ---------------------------------------------------------------------------
// Parameter decode (Sec. II.B): x = [D0, alpha, r0, beta, n, h] with S = 2,
// so lambda = 2 alpha, mu = alpha, f_R = D0 e^{-2 alpha (r - r0)},
// f_A = 2 D0 e^{-alpha (r - r0)}.  A candidate outside the potential's domain
// is replaced by a harmless stand-in so the arithmetic stays finite; its
// outputs are set to NaN by the finalize kernels.
// ---------------------------------------------------------------------------
// Parameter vectors: minimal [D0, alpha, r0, beta, n, h]; Tersoff form
// [D0, alpha, r0, S, gamma, n, c, d, h].
template <bool Full>
struct Form {
    static constexpr int nx = Full ? 9 : 6;
};

template <bool Full>
__device__ __forceinline__ bool params_valid(const double* __restrict__ x) {
    bool fin = true;
#pragma unroll
    for (int k = 0; k < Form<Full>::nx; ++k) fin = fin && isfinite(x[k]);
    if constexpr (Full) {
        return fin && x[0] > 0.0 && x[1] > 0.0 && x[3] > 1.0 && x[4] >= 0.0 && x[5] > 0.0 &&
               x[7] != 0.0;
    } else {
        return fin && x[0] > 0.0 && x[1] > 0.0 && x[4] > 0.0 && x[3] >= 0.0;
    }
}

// x -> the record of the form-independent site routine.  The minimal form leaves
// the Tersoff form's fields unwritten.
template <typename S, bool Full>
__device__ __forceinline__ void decode_record(const double* __restrict__ x, Rec<S>& o) {
    const double log2e = 1.4426950408889634;
    const bool ok = params_valid<Full>(x);
    double D0 = x[0], al = x[1], r0 = x[2], n, h;
    if constexpr (Full) {
        double Sl = x[3], gam = x[4], c = x[6], d = x[7];
        n = x[5];
        h = x[8];
        if (!ok) { D0 = 3.0; al = 1.4; r0 = 2.2; Sl = 2.0; gam = 0.3; n = 0.6; c = 1.0; d = 1.0; h = -0.6; }
        const double mu = al * sqrt(2.0 / Sl), lam = al * sqrt(2.0 * Sl);
        o.aA64 = mu * log2e;
        o.aR64 = lam * log2e;
        o.DR64 = D0 / (Sl - 1.0);
        o.DA64 = Sl * D0 / (Sl - 1.0);
        o.aR = (S)o.aR64;
        o.DA = (S)o.DA64;
        o.zs = S(1);
        o.ccs = S(0.5);
        o.hmu = (S)(0.5 * mu);
        o.hlambda = (S)(0.5 * lam);
        const double K = gam * c * c / (d * d);
        o.gam = (S)gam;
        o.K = (S)K;
        // where d^2 overflows, the largest value: g^T = gamma then, and no
        // product with rho = 1/(d^2 + t^2) is infinity times 0
        o.d2 = (S)(sizeof(S) == 4 ? fmin(d * d, 3.4028234663852886e38) : fmin(d * d, kMaxDouble));
        o.Kd2 = (S)(K * d * d);
    } else {
        // S = 2: mu = alpha, lambda = 2 alpha, DR = D0, DA = 2 D0
        double be = x[3];
        n = x[4];
        h = x[5];
        if (!ok) { D0 = 3.0; al = 1.4; r0 = 2.2; be = 0.3; n = 0.6; h = -0.6; }
        o.aA64 = al * log2e;
        o.DR64 = D0;
        o.DA = (S)(2.0 * D0);
        o.zs = (S)be;
        o.ccs = (S)(0.5 * be);
        o.hmu = (S)(0.5 * al);
    }
    o.r0 = r0;
    o.ninv2n64 = -1.0 / (2.0 * n);
    o.aA = (S)o.aA64;
    o.DR = (S)o.DR64;
    o.n = (S)n;
    o.ninv2n = (S)o.ninv2n64;
    o.h = (S)h;
    o.hlo = (S)(h - (double)o.h);
    o.valid = ok ? S(1) : S(0);
}

template <typename S>
struct alignas(4 * sizeof(S)) Vec4 {
    S x, y, z, w;
};

template <typename S>
struct BArgs {
    SetDev set;
    const Item* items;
    const int* bin_off;       // null: one item per block
    const double* x;          // [P][6] (minimal) or [P][9] (Tersoff form) parameter sets
    double* partial;          // [P][nslots][nv]
    int nv;
    // MODE_EVAL outputs (caller numbering); may be null
    double* force;            // [P][3][N]
    double* atom_virial;      // [P][9][N]
    const double* vel;        // [3][N]
    // MODE_EVAL without a finalize kernel: the totals go straight to energy
    // [P][S] and virial [P][S][6] (either may be null)
    int direct;
    double* energy;
    double* virial;
    double* heat;             // [P][3], two-pass evaluation of a set of one structure
    // adjoint inputs
    const double* coef;       // [P][S][8]
    // force residuals F - F* of the batched atoms, [P][3][N] (sorted atom
    // order): written by the fitness kernel when non-null, read by the adjoint
    S* resid;
};

template <typename S>
__device__ __forceinline__ GeomArrays<S> geom_of(const SetDev& d);
template <>
__device__ __forceinline__ GeomArrays<float> geom_of<float>(const SetDev& d) { return d.gf; }
template <>
__device__ __forceinline__ GeomArrays<double> geom_of<double>(const SetDev& d) { return d.gd; }
template <typename S>
__device__ __forceinline__ const S* fref_of(const SetDev& d);
template <>
__device__ __forceinline__ const float* fref_of<float>(const SetDev& d) { return d.fref32; }
template <>
__device__ __forceinline__ const double* fref_of<double>(const SetDev& d) { return d.fref64; }

struct ItemCtx {
    int s, a0, Ns, npad, R, q, la, atom, steps, slot, g, xsz, own, Mw, unit, wpr;
    bool active, block_sync;
};

__device__ __forceinline__ ItemCtx item_ctx(const SetDev& d, const Item& it) {
    // Item fields are uniform across the block; npad is 8, 16, 32, 64 or a
    // multiple of 64, so lane -> (replica, atom) needs no vector division.
    // (Plain variables until the end: a struct written in the branches stays in
    // scratch, and every use of a field is a load then.)
    const int tid = threadIdx.x, R = it.R, npad = it.npad;
    const bool one = npad <= 64;
    const int sh = 31 - __clz(npad);
    const int waves = npad >> 6;                           // wavefronts per replica above 64
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = blockDim.x >> 6;
    // A structure's chunks of 64 atoms get cheaper in order (atoms are
    // sorted by coordination), and wavefront w of a block runs on SIMD
    // w mod 4: rows of four wavefronts take the (chunk, replica) pairs in
    // turn from either end, so that no SIMD collects the costly chunks of
    // several rows while the block waits for it at the exchange (M <= 12
    // launch of 500 candidates x 101 packings: 765 us in plain order, 712 us).
    const int row = wid & ~3, in_row = (nw - row) < 4 ? nw - row : 4;
    const int rank = (row & 4) ? row + in_row - 1 - (wid - row) : wid;
    const int chunk = rank / R;                            // scalar division
    const bool in = chunk < waves;
    ItemCtx x;
    x.s = it.s;
    x.a0 = it.a0;
    x.Ns = it.ns;
    x.npad = npad;
    x.R = R;
    x.unit = one ? 0 : rank;
    x.wpr = one ? 1 : waves;
    x.g = one ? npad : 64;
    x.q = one ? tid >> sh : in ? rank - chunk * R : R;
    x.la = one ? tid & (npad - 1) : (in ? chunk << 6 : 0) + (tid & 63);
    x.active = (x.q < x.R) && (x.la < x.Ns);
    x.atom = x.a0 + (x.active ? x.la : 0);
    x.steps = (it.nc + x.R - 1) / x.R;
    x.slot = it.slot;
    x.xsz = it.xsz;
    x.block_sync = npad > 64;
    // own exchange slot base: the first chunk's slots start at 0, and a chunk's
    // first atom is always a real atom
    const int chunk0 = one ? 0 : __builtin_amdgcn_readfirstlane(x.la & ~63);
    x.own = x.q < x.R ? (chunk0 ? d.xbase[x.a0 + chunk0] : 0) + (x.la - chunk0) + x.q * x.xsz : 0;
    // the wavefront's largest coordination is that of its first atom (sorted);
    // -1: no replica here (whole wavefronts past the last replica)
    x.Mw = __builtin_amdgcn_readfirstlane(x.q) >= x.R ? -1 : d.nnb[x.a0 + chunk0];
    return x;
}

// LDS ordering: a replica inside one wavefront only needs the compiler not to
// move LDS accesses across this point; larger replicas need the block barrier.
__device__ __forceinline__ void exchange_sync(bool block) {
    if (block) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// One structure total of candidate c: value k of the partial-sum slot, or, for
// an evaluation that needs no more, the energy or virial itself.
template <int MODE, typename S>
__device__ __forceinline__ void put_sum(const BArgs<S>& A, const ItemCtx& x, int c, int k, double sum, bool valid) {
    if (MODE == MODE_EVAL && A.direct) {
        const double v = valid ? sum : __longlong_as_double(0x7ff8000000000000ll);
        const size_t cs = (size_t)c * A.set.S + x.s;
        if (k == 0 && A.energy) A.energy[cs] = v;
        if (k >= 1 && k <= 6 && A.virial) A.virial[cs * 6 + k - 1] = v;
    } else {
        A.partial[((size_t)c * A.set.nslots + x.slot) * A.nv + k] = sum;
    }
}

// Sum v[0..7] over the lane group.  A replica inside one wavefront is done
// (put_sum); the wavefronts of a larger one leave their sums, values off ..
// off + 7 of those in wmask, in red[unit] for flush_sums.  GF is the group size
// when known at compile time (0: x.g at run time).
template <int MODE, int NV, int GF = 0, int SYNC = -1, typename S>
__device__ __forceinline__ void store_group(double* v, const BArgs<S>& A, const ItemCtx& x, bool group_ok, int c,
                                            int off, int wmask, bool valid, double* __restrict__ red) {
    int vidx;
    const double sum = GF ? group_reduce8_t<(GF ? GF : 64)>(v, &vidx) : group_reduce8(v, x.g, &vidx);
    const int lane = threadIdx.x & 63;
    if ((lane & ((x.g >> 3) - 1)) == 0 && ((wmask >> vidx) & 1)) {
        if (SYNC < 0 ? x.block_sync : SYNC == 1) red[x.unit * NV + off + vidx] = sum;
        else if (group_ok) put_sum<MODE>(A, x, c, off + vidx, sum, valid);
    }
}

// Total of a structure of several wavefronts for candidate c: the wavefronts'
// sums in chunk order, by the replica's last (cheapest) wavefront.  Called one
// block barrier after the store_group that left them, and one before the next.
template <int MODE, int NV, typename S>
__device__ __forceinline__ void flush_sums(const BArgs<S>& A, const ItemCtx& x, int c, int nval, bool valid,
                                           const double* __restrict__ red) {
    const int lane = threadIdx.x & 63;
    if (x.unit / x.R != x.wpr - 1 || lane >= nval) return;
    double t = 0.0;
    for (int w = 0; w < x.wpr; ++w) t += red[(w * x.R + x.q) * NV + lane];
    put_sum<MODE>(A, x, c, lane, t, valid);
}

// LDS layout of a block while it works on an item: [kRedBytes of wavefront
// sums][it.nc parameter records][R x xsz exchange slots (Vec4); adjoint: R x npad force residuals
// (Vec4) instead].  The exchange follows the item's own records, so the LDS a launch
// gets for the largest (records + exchange) of its structures covers every
// item, whatever the candidate tiles of the other structures in the launch.
template <typename S>
__device__ __forceinline__ size_t lds_param_bytes(int nc) {
    return ((size_t)nc * sizeof(Rec<S>) + 31) & ~(size_t)31;
}

// The moment path's two values per bond wait in the bond's own exchange slot
// until its gradient takes their place: nobody reads the slot in between.
template <typename S>
struct ParkSlots {
    Vec4<S>* own;
    int g;
    __device__ __forceinline__ void put(int j, S x, S y) const {
        own[j * g].x = x;
        own[j * g].y = y;
    }
    __device__ __forceinline__ void get(int j, S& x, S& y) const {
        x = own[j * g].x;
        y = own[j * g].y;
    }
};

// SYNC: 1 the replicas span several wavefronts, 0 each lies inside one, -1 known
// at run time only (x.block_sync).
// Resid (fitness mode): also write each atom's force residual to A.resid (the
// gradient's fitness call; a separate instance, so the fitness alone carries
// no trace of it).
template <typename S, int MODE, int M, int GF = 0, int SYNC = -1, bool Full = false, bool Resid = false>
__device__ __forceinline__ void run_batched(const BArgs<S>& A, const Item& it, const ItemCtx& x,
                                            unsigned char* __restrict__ lds) {
    const SetDev& d = A.set;
    const int N = d.N;
    constexpr int NV = MODE == MODE_FIT ? kNVFit : kNVEval;
    const bool sync = SYNC < 0 ? x.block_sync : SYNC == 1;
    double* __restrict__ red = reinterpret_cast<double*>(lds - kRedBytes);
    const Rec<S>* __restrict__ pbuf = reinterpret_cast<const Rec<S>*>(lds);
    Vec4<S>* __restrict__ xb = reinterpret_cast<Vec4<S>*>(lds + lds_param_bytes<S>(it.nc));
    constexpr bool Mom = MODE != MODE_EVAL;
    Geo<S, M, Full, Mom> g;
    g.load(d, x.atom, x.active);
    constexpr int MM = M > 0 ? M : 1;
    int rv[MM];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        rv[m] = d.rev[(size_t)m * N + x.atom] + x.q * x.xsz;
        g.rows_apart();
    }
#pragma unroll
    for (int m = 0; m < M; ++m) rv[m] = x.active ? rv[m] : x.own + m * x.g;
    const S* fr = fref_of<S>(d);
    S frx = S(0), fry = S(0), frz = S(0);
    if (MODE == MODE_FIT) {
        const S a = fr[x.atom], b = fr[(size_t)N + x.atom], c = fr[(size_t)2 * N + x.atom];
        frx = x.active ? a : S(0); fry = x.active ? b : S(0); frz = x.active ? c : S(0);
    }
    const int orig = d.perm[x.atom];
    S vx = S(0), vy = S(0), vz = S(0);
    if (MODE == MODE_EVAL && A.vel) {
        vx = (S)A.vel[orig]; vy = (S)A.vel[(size_t)N + orig]; vz = (S)A.vel[(size_t)2 * N + orig];
    }
    __syncthreads();                                   // the records
    // the structure totals of a step, once its wavefronts' sums are all there
    auto flush = [&](int step) __attribute__((always_inline)) {
        const int cl = x.q + step * x.R;
        if (cl < it.nc)
            flush_sums<MODE, NV>(A, x, it.c0 + cl, MODE == MODE_FIT ? 8 : 11, pbuf[cl].valid != S(0), red);
    };

    for (int step = 0; step < x.steps; ++step) {
        const int cl = x.q + step * x.R;
        const bool group_ok = cl < it.nc;
        const bool cok = x.active && group_ok;
        const int clv = group_ok ? cl : 0;
        const int c = it.c0 + clv;
        Cand<S, Full> p;
        load_cand(pbuf[clv], p);
        // Each bond gradient G_j goes to its exchange slot as soon as the site
        // routine emits it and is folded into this atom's own force sum and
        // the virial, so no bond-gradient array stays live across the exchange.
        double U;
        S Fx = S(0), Fy = S(0), Fz = S(0);
        S w6[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) w6[k] = S(0);
        site_eval_sink<S, M, true, (M > kPairwiseMax<S, Full, Mom>), Full, true, Mom>(
            g, p, U, [&](int m, S gx, S gy, S gz) {
                S* slot = &xb[x.own + m * x.g].x;     // the fourth component is never read
                slot[0] = gx;
                slot[1] = gy;
                slot[2] = gz;
                Fx += gx; Fy += gy; Fz += gz;
                const S rm = g.length(m), dx = rm * g.ux[m], dy = rm * g.uy[m], dz = rm * g.uz[m];
                w6[0] -= dx * gx; w6[1] -= dy * gy; w6[2] -= dz * gz;
                w6[3] -= dy * gz; w6[4] -= dz * gx; w6[5] -= dx * gy;
            },
            ParkSlots<S>{xb + x.own, x.g});
        exchange_sync(sync);
        if (sync && step > 0) flush(step - 1);
        S wi[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) wi[k] = S(0);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const Vec4<S> r = xb[rv[m]];
            Fx -= r.x;
            Fy -= r.y;
            Fz -= r.z;
            if (MODE == MODE_EVAL) {
                const S rm = g.length(m), dx = rm * g.ux[m], dy = rm * g.uy[m], dz = rm * g.uz[m];
                wi[0] += dx * r.x; wi[1] += dx * r.y; wi[2] += dx * r.z;
                wi[3] += dy * r.x; wi[4] += dy * r.y; wi[5] += dy * r.z;
                wi[6] += dz * r.x; wi[7] += dz * r.y; wi[8] += dz * r.z;
            }
        }
        exchange_sync(sync);
        // Lanes outside the structure have f_C = 0 and zero reference forces, so
        // their energy, virial and residual are exactly zero.
        double v[8];
        v[0] = (double)U;
#pragma unroll
        for (int k = 0; k < 6; ++k) v[1 + k] = (double)w6[k];
        if (MODE == MODE_FIT) {
            const S ax = Fx - frx, ay = Fy - fry, az = Fz - frz;
            v[7] = (double)(ax * ax + ay * ay + az * az);
            if (Resid && cok) {
                S* r = A.resid + (size_t)c * 3 * N;
                r[x.atom] = ax;
                r[(size_t)N + x.atom] = ay;
                r[(size_t)2 * N + x.atom] = az;
            }
            store_group<MODE, NV, GF, SYNC>(v, A, x, group_ok, c, 0, 0xff, true, red);
        } else {
            v[7] = 0.0;
            store_group<MODE, NV, GF, SYNC>(v, A, x, group_ok, c, 0, 0xff, p.valid != S(0), red);
            double u[8];
            const S jx = wi[0] * vx + wi[1] * vy + wi[2] * vz;
            const S jy = wi[3] * vx + wi[4] * vy + wi[5] * vz;
            const S jz = wi[6] * vx + wi[7] * vy + wi[8] * vz;
            u[0] = (double)jx;
            u[1] = (double)jy;
            u[2] = (double)jz;
            u[3] = u[4] = u[5] = u[6] = u[7] = 0.0;
            store_group<MODE, NV, GF, SYNC>(u, A, x, group_ok, c, 8, 0x07, p.valid != S(0), red);
            if (cok && A.force) {
                double* f = A.force + (size_t)c * 3 * N;
                f[orig] = (double)Fx;
                f[(size_t)N + orig] = (double)Fy;
                f[(size_t)2 * N + orig] = (double)Fz;
            }
            if (cok && A.atom_virial) {
                double* w = A.atom_virial + (size_t)c * 9 * N;
#pragma unroll
                for (int k = 0; k < 9; ++k) w[(size_t)k * N + orig] = (double)wi[k];
            }
        }
    }
    if (sync) {
        __syncthreads();
        flush(x.steps - 1);
    }
}

__device__ __forceinline__ void run_idle(int barriers) {
    __syncthreads();                                   // the records
    for (int b = 0; b < barriers; ++b) __syncthreads();
}

// Call f(integral_constant<M>) for the variant that serves coordination m.
template <int LO, int HI, typename F>
__device__ __forceinline__ void dispatch_m(int m, F&& f) {
    if constexpr (LO >= HI) {
        f(std::integral_constant<int, HI>{});
    } else {
        if (m <= LO) f(std::integral_constant<int, LO>{});
        else dispatch_m<LO + 1, HI>(m, f);
    }
}

// Lowest compiled variant of a class; the exchange-slot layout of a set
// reserves at least three slots per atom, so every class can run any structure.
template <int MC>
struct ClassLo {
    static constexpr int value = MC <= 4 ? 0 : 3;
};

// Decode the item's parameter sets into the LDS records (all threads take part).
// The block synchronises after its wavefronts have issued their geometry loads
// (run_batched, run_adjoint, run_idle), so one memory round trip covers both.
template <typename S, bool Full = false>
__device__ __forceinline__ void decode_item(const BArgs<S>& A, const Item& it, unsigned char* lds) {
    Rec<S>* pbuf = reinterpret_cast<Rec<S>*>(lds);
    for (int t = threadIdx.x; t < it.nc; t += blockDim.x)
        decode_record<S, Full>(A.x + Form<Full>::nx * (size_t)(it.c0 + t), pbuf[t]);
}

template <typename S, int MODE, int MC, bool Full, bool Resid = false>
__device__ __forceinline__ void batched_item(const BArgs<S>& A, const Item& it, unsigned char* lds) {
    const ItemCtx x = item_ctx(A.set, it);
    decode_item<S, Full>(A, it, lds);
    const int Mw = x.Mw;
    if (Mw < 0) {
        // whole wavefront outside every replica; replicas of several wavefronts
        // synchronise the block twice per step and once at the end
        run_idle(x.block_sync ? 2 * x.steps + 1 : 0);
        return;
    }
    dispatch_m<ClassLo<MC>::value, MC>(Mw, [&](auto mv) {
        // the float fitness kernel of the minimal potential gets copies for
        // structures of several wavefronts and (M <= 4) of one: with the group
        // size and the kind of exchange fixed at compile time the reduction
        // needs no branches and no copies around the in-place lane swaps
        if constexpr (MODE == MODE_FIT && sizeof(S) == 4 && !Full) {
            if (x.block_sync) {
                run_batched<S, MODE, decltype(mv)::value, 64, 1, Full, Resid>(A, it, x, lds);
                return;
            }
            if constexpr (MC <= 4) {
                if (x.g == 64) {
                    run_batched<S, MODE, decltype(mv)::value, 64, 0, Full, Resid>(A, it, x, lds);
                    return;
                }
            }
            run_batched<S, MODE, decltype(mv)::value, 0, 0, Full, Resid>(A, it, x, lds);
            return;
        }
        run_batched<S, MODE, decltype(mv)::value, 0, -1, Full, Resid>(A, it, x, lds);
    });
}

// Occupancy target per class: the float fitness kernel of the M <= 4 class
// fits 4 wavefronts per SIMD (128 registers).
template <typename S, int MODE, int MC>
struct WavesPerEU {
    static constexpr int value = (MC <= 4 && sizeof(S) == 4 && MODE == MODE_FIT) ? 4 : 1;
};

// The item, uniform across the block, in scalar registers: work lists do not change
// while a kernel runs.
__device__ __forceinline__ Item load_item(const Item* p) {
    const auto* c = (const __attribute__((address_space(4))) Item*)p;
    Item it;
    it.s = c->s; it.c0 = c->c0; it.nc = c->nc; it.cost = 0;
    it.a0 = c->a0; it.ns = c->ns; it.npad = c->npad; it.slot = c->slot; it.xsz = c->xsz; it.R = c->R;
    return it;
}

template <typename S, int MODE, int MC, bool Full = false, bool Resid = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(WavesPerEU<S, MODE, MC>::value)))
void k_batched(BArgs<S> A) {
    extern __shared__ __align__(32) unsigned char lds_raw[];
    // without bins, block b has item b
    const int b0 = A.bin_off ? A.bin_off[blockIdx.x] : (int)blockIdx.x;
    const int b1 = A.bin_off ? A.bin_off[blockIdx.x + 1] : b0 + 1;
    for (int i = b0; i < b1; ++i) {
        const Item it = load_item(A.items + i);
        batched_item<S, MODE, MC, Full, Resid>(A, it, lds_raw + kRedBytes);
        __syncthreads();
    }
}

// The plain schedule: one launch per (candidate, structure), a single block
// that evaluates the item A.items[0].  The same device code as k_batched,
// under a kernel name of its own so that profiles keep the two apart.
template <typename S, int MODE, int MC, bool Full = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(WavesPerEU<S, MODE, MC>::value)))
void k_plain(BArgs<S> A) {
    extern __shared__ __align__(32) unsigned char lds_raw[];
    batched_item<S, MODE, MC, Full>(A, load_item(A.items), lds_raw + kRedBytes);
}

// ---------------------------------------------------------------------------
// Adjoint kernel: dZ/dx of the fitness.  For candidate c and structure s,
//   dZ/dx|_s = sum_i [ k_e U_i' - sum_j G_ij' . delta_ij ],
//   delta_ij = k_f (a_j - a_i) + C_s r_ij,   a = F - F*,
// where ' is the derivative with respect to the parameters (six, or nine for
// the Tersoff form), k_e = w_e (e_s - e*_s)/(N_s Z_e Q_e), k_f = w_f/(Z_f Q_f) and
// C_s = w_v/(N_s Z_v Q_v) times the symmetric matrix of virial residuals (off
// diagonals halved).  These follow from dF_i/dx = -d/dx dE/dr_i and
// dW/dx = -sum r_ij (x) dG_ij/dx.
//
// sum_j G_ij . delta_ij is the derivative D of U_i when every bond vector moves
// along its delta_ij, so the contraction is L[U_i'] with the linear map
// L[f] = k_e f - D f.  U_i' is a closed form in each bond's r, f_C and angular
// sums, so one derivative along delta of those few quantities serves all the
// parameters: no bond gradient is formed, and the parameter count does not
// multiply the pair loop.  Against forward-mode duals over three to six
// parameters at a time through the whole gradient (256 registers, 2 KB of
// scratch a lane at M = 12, bound by VALU issue and spills): a fitness_grad call
// on 300 structures of 8-512 atoms x 64 candidates 1415 -> 450 us (float32), on
// 18 structures x 5 Tersoff-form candidates 1004 -> 288 us (float64).
// ---------------------------------------------------------------------------

// The sums over an atom's bonds that dZ/dx is made of, each under L; the
// parameters' own factors (D0, mu, ...) are the same for every atom and are
// applied once per candidate in float64 (k_finalize_grad).  With
// e_R = e^{-lambda (r - r0)}, e_A = e^{-mu (r - r0)}, Y = -1/2 f_C e_A db/dzeta:
//   R, A     f_C e_R,  f_C b e_A
//   DR, DA   the same times r - r0
//   N        -1/2 f_C e_A db/dn
//   minimal: Z2 = Y sum_k f_C t^2, Z1 = Y sum_k f_C t        (t = cos - h)
//   Tersoff: S0 = Y sum_k f_C, SQ = Y sum_k f_C q, SQR = Y sum_k f_C q rho,
//            SP = Y sum_k f_C t rho^2   (rho = 1/(d^2 + t^2), q = t^2 rho)
enum GradSum {
    GS_R = 0, GS_A, GS_DR, GS_DA, GS_N,
    GS_Z2, GS_Z1,
    GS_S0 = 5, GS_SQ, GS_SQR, GS_SP
};
template <bool Full>
struct GradSums {
    static constexpr int value = Full ? 9 : 7;
};

// Largest coordination whose angular sums without moments take every
// unordered pair once, with the sums of all bonds live; above it they are
// formed bond by bond.
template <typename S>
constexpr int kAdjointPairs = sizeof(S) == 8 ? 4 : 12;

// One atom's grad sums.  rec: the candidate's decoded record, (ax, ay, az) this
// atom's force residual, aj(m) the residual of the atom at the far end of bond
// m, cf the coefficients k_e, k_f, C_s (xx yy zz yz zx xy, off-diagonals halved)
// of the (candidate, structure).
template <typename S, int M, bool Full, typename Aj>
__device__ __forceinline__ void adjoint_sums(Geo<S, M, Full>& g, const Rec<S>& rec, S ax, S ay, S az,
                                             Aj&& aj, const double* __restrict__ cf,
                                             S (&L)[GradSums<Full>::value]) {
    constexpr int MM = M > 0 ? M : 1;
    const S ke = (S)cf[0], kf = (S)cf[1];
    const S cxx = (S)cf[2], cyy = (S)cf[3], czz = (S)cf[4];
    const S cyz = (S)cf[5], czx = (S)cf[6], cxy = (S)cf[7];
    Cand<S, Full> p;
    load_cand(rec, p);
    // keep the float copies of r and the uncached cos(theta) out of registers
    // across candidates
    if constexpr (sizeof(S) == 4 && M > 0) opaque(g.r);
    if constexpr (!Geo<S, M, Full>::kCache && M > 1) {
        opaque(g.ux);
        opaque(g.uy);
        opaque(g.uz);
    }
    // D of bond m's length, f_C and unit vector
    struct BondD {
        S dr, dfc, wx, wy, wz;
    };
    auto bond_d = [&](int m) __attribute__((always_inline)) {
        const Vec4<S> a = aj(m);
        const S rm = g.length(m), dx = rm * g.ux[m], dy = rm * g.uy[m], dz = rm * g.uz[m];
        const S ex = kf * (a.x - ax) + cxx * dx + cxy * dy + czx * dz;
        const S ey = kf * (a.y - ay) + cxy * dx + cyy * dy + cyz * dz;
        const S ez = kf * (a.z - az) + czx * dx + cyz * dy + czz * dz;
        BondD d;
        d.dr = ex * g.ux[m] + ey * g.uy[m] + ez * g.uz[m];
        d.dfc = (S(2) * g.hfcp[m]) * d.dr;
        d.wx = (ex - d.dr * g.ux[m]) * g.rinv[m];
        d.wy = (ey - d.dr * g.uy[m]) * g.rinv[m];
        d.wz = (ez - d.dr * g.uz[m]) * g.rinv[m];
        return d;
    };
    // Angular sums over the other bonds and their D.  Minimal: s[0] = sum f_C t^2,
    // s[1] = sum f_C t.  Tersoff: sums of f_C, f_C q, f_C q rho, f_C t rho^2.
    constexpr int NS = Full ? 4 : 2;
    auto terms = [&](S t, S dt, S (&f)[NS], S (&df)[NS]) __attribute__((always_inline)) {
        if constexpr (Full) {
            const S t2 = t * t;
            const S rho = drcp(p.d2 + t2);
            const S q = t2 * rho, pr = t * rho * rho;
            f[0] = S(1); f[1] = q; f[2] = q * rho; f[3] = pr;
            const S e = S(2) * pr * dt;           // -D rho
            df[0] = S(0); df[1] = p.d2 * e; df[2] = (p.d2 * rho - q) * e;
            df[3] = (rho * rho) * (S(1) - S(4) * q) * dt;
        } else {
            f[0] = t * t; f[1] = t;
            df[0] = (S(2) * t) * dt; df[1] = dt;
        }
    };
    const S mu = S(2) * p.hmu, lam = S(2) * p.hlambda;
    const S c1 = S(2) * p.ninv2n * p.ninv2n;              // 1 / (2 n^2)
    const S ln2 = S(0.6931471805599453);
#pragma unroll
    for (int k = 0; k < GradSums<Full>::value; ++k) L[k] = S(0);
    auto bond = [&](int j, S drj, S dfcj, const S (&s)[NS], const S (&ds)[NS]) __attribute__((always_inline)) {
        S z, dz;
        if constexpr (Full) {
            z = p.gam * s[0] + p.K * s[1];
            dz = p.gam * ds[0] + p.K * ds[1];
        } else {
            z = p.zs * s[0];
            dz = p.zs * ds[0];
        }
        // zeta = 0: b = 1 and every derivative of b is dropped (zn = 0)
        const bool pos = z > S(0);
        const S zsafe = pos ? z : S(1);
        const S delta = (S)(g.r[j] - p.r0);
        const S eA = dexp2(-(p.aA * delta));
        S eR;
        if constexpr (Full) eR = dexp2(-(p.aR * delta));
        else eR = eA * eA;
        const S l2z = dlog2(zsafe);
        const S zne = dexp2(p.n * l2z);       // formed before the selection: no branch
        const S zn = pos ? zne : S(0);
        const S onep = S(1) + zn;
        const S v = drcp(onep), w = zn * v, iz = drcp(zsafe);
        const S l2p = dlog2(onep);
        const S b = dexp2(p.ninv2n * l2p);
        // db/dzeta, db/dn (over b: kn) and their D, with e = D zeta / zeta:
        // D w = n w v e, D(db/dn) = Db (kn + v ln zeta)
        const S e = dz * iz;
        const S db = S(-0.5) * (b * w) * e;
        const S bz = S(-0.5) * (b * w) * iz;
        const S dbz = (bz * e) * (p.n * v - S(0.5) * w - S(1));
        const S kn = ln2 * (c1 * l2p + p.ninv2n * (w * l2z));
        const S bn = b * kn;
        const S dbn = db * (kn + (v * ln2) * l2z);
        const S R = g.fc[j] * eR, dR = dfcj * eR - (lam * drj) * R;
        const S q = g.fc[j] * eA, dq = dfcj * eA - (mu * drj) * q;
        const S A = b * q, dA = b * dq + db * q;
        const S LR = ke * R - dR, LA = ke * A - dA;
        L[GS_R] += LR;
        L[GS_A] += LA;
        L[GS_DR] += delta * LR - drj * R;
        L[GS_DA] += delta * LA - drj * A;
        L[GS_N] -= S(0.5) * (ke * (q * bn) - (dq * bn + q * dbn));
        const S Y = S(-0.5) * (q * bz), dY = S(-0.5) * (dq * bz + q * dbz);
        const S LY = ke * Y - dY;
#pragma unroll
        for (int c = 0; c < NS; ++c) L[5 + c] += LY * s[c] - Y * ds[c];
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (Geo<S, M, Full>::kMoments) {
        // Float minimal form, larger coordination: the pair sums from the moments
        // sum f_C, sum f_C u, sum f_C u u^T and their D, so the work grows with
        // the bonds, not the bond pairs, and nothing is held per bond.
        S exx = S(0), eyy = exx, ezz = exx, eyz = exx, ezx = exx, exy = exx, nx = exx, ny = exx, nz = exx;
        S dS = S(0);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const BondD d = bond_d(m);
            const S ux = g.ux[m], uy = g.uy[m], uz = g.uz[m], f = g.fc[m];
            // D(f u u^T) = v u^T + u v^T with v = f w + dfc u / 2
            const S gx = f * d.wx, gy = f * d.wy, gz = f * d.wz, hf = S(0.5) * d.dfc;
            const S vx = gx + hf * ux, vy = gy + hf * uy, vz = gz + hf * uz;
            nx += gx + d.dfc * ux; ny += gy + d.dfc * uy; nz += gz + d.dfc * uz;
            exx += (S(2) * vx) * ux; eyy += (S(2) * vy) * uy; ezz += (S(2) * vz) * uz;
            eyz += vy * uz + vz * uy; ezx += vz * ux + vx * uz; exy += vx * uy + vy * ux;
            dS += d.dfc;
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const BondD d = bond_d(j);
            const S ux = g.ux[j], uy = g.uy[j], uz = g.uz[j];
            const S yx = g.txx * ux + g.txy * uy + g.tzx * uz, yy = g.txy * ux + g.tyy * uy + g.tyz * uz,
                    yz = g.tzx * ux + g.tyz * uy + g.tzz * uz;
            const S zx = exx * ux + exy * uy + ezx * uz, zy = exy * ux + eyy * uy + eyz * uz,
                    zz = ezx * ux + eyz * uy + ezz * uz;
            // D of sum_k f_C c and sum_k f_C c^2 over the other bonds (c = 1 for
            // the bond itself)
            const S p1 = (d.wx * g.mx + d.wy * g.my + d.wz * g.mz) + (ux * nx + uy * ny + uz * nz) - d.dfc;
            const S p2 = S(2) * (d.wx * yx + d.wy * yy + d.wz * yz) + (ux * zx + uy * zy + uz * zz) - d.dfc;
            const S ds0 = dS - d.dfc;
            const S t = (g.sh[j] - p.h) - p.hlo;
            const S s1 = g.ss[j] * t;
            const S s[NS] = {g.sv[j] + s1 * t, s1};
            const S ds[NS] = {p2 - p.h * (S(2) * p1 - p.h * ds0), p1 - p.h * ds0};
            bond(j, d.dr, d.dfc, s, ds);
        }
    } else if constexpr (M <= kAdjointPairs<S>) {
        // every unordered bond pair once
        BondD d[MM];
#pragma unroll
        for (int m = 0; m < M; ++m) d[m] = bond_d(m);
        S s[MM][NS], ds[MM][NS];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int k = 0; k < NS; ++k) s[m][k] = ds[m][k] = S(0);
        int pidx = 0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
#pragma unroll
            for (int k = j + 1; k < M; ++k) {
                const S t = (g.cosjk(j, k, pidx++) - p.h) - p.hlo;
                const S dt = (d[j].wx * g.ux[k] + d[j].wy * g.uy[k] + d[j].wz * g.uz[k]) +
                             (d[k].wx * g.ux[j] + d[k].wy * g.uy[j] + d[k].wz * g.uz[j]);
                S f[NS], df[NS];
                terms(t, dt, f, df);
#pragma unroll
                for (int c = 0; c < NS; ++c) {
                    s[j][c] += g.fc[k] * f[c];
                    s[k][c] += g.fc[j] * f[c];
                    ds[j][c] += d[k].dfc * f[c] + g.fc[k] * df[c];
                    ds[k][c] += d[j].dfc * f[c] + g.fc[j] * df[c];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < M; ++j) bond(j, d[j].dr, d[j].dfc, s[j], ds[j]);
    } else {
        // one bond at a time, every pair from both ends: twice the pair
        // arithmetic, but the sums of one bond only are live
        BondD d[MM];
#pragma unroll
        for (int m = 0; m < M; ++m) d[m] = bond_d(m);
#pragma unroll
        for (int j = 0; j < M; ++j) {
            S s[NS], ds[NS];
#pragma unroll
            for (int c = 0; c < NS; ++c) s[c] = ds[c] = S(0);
#pragma unroll
            for (int k = 0; k < M; ++k) {
                if (k == j) continue;
                const S t = ((g.ux[j] * g.ux[k] + g.uy[j] * g.uy[k] + g.uz[j] * g.uz[k]) - p.h) - p.hlo;
                const S dt = (d[j].wx * g.ux[k] + d[j].wy * g.uy[k] + d[j].wz * g.uz[k]) +
                             (d[k].wx * g.ux[j] + d[k].wy * g.uy[j] + d[k].wz * g.uz[j]);
                S f[NS], df[NS];
                terms(t, dt, f, df);
#pragma unroll
                for (int c = 0; c < NS; ++c) {
                    s[c] += g.fc[k] * f[c];
                    ds[c] += d[k].dfc * f[c] + g.fc[k] * df[c];
                }
            }
            bond(j, d[j].dr, d[j].dfc, s, ds);
        }
    }
}

// dZ/dx from the totals T of the grad sums: the parameters' factors.
template <bool Full>
__device__ __forceinline__ void grad_from_sums(const double* __restrict__ x, const double* __restrict__ T,
                                               double* __restrict__ G) {
    const double D0 = x[0], al = x[1];
    if constexpr (Full) {
        // DR = D0/(S-1), DA = S DR, mu = alpha sqrt(2/S), lambda = alpha sqrt(2S)
        const double Sl = x[3], gam = x[4], c = x[6], d = x[7];
        const double sm1 = Sl - 1.0, DR = D0 / sm1, DA = Sl * DR;
        const double rs = sqrt(2.0 / Sl), rl = sqrt(2.0 * Sl), mu = al * rs, lam = al * rl;
        const double K = gam * c * c / (d * d);
        G[0] = 0.5 * (T[GS_R] - Sl * T[GS_A]) / sm1;
        G[1] = 0.5 * (rs * DA * T[GS_DA] - rl * DR * T[GS_DR]);
        G[2] = 0.5 * (lam * DR * T[GS_R] - mu * DA * T[GS_A]);
        G[3] = 0.5 * ((DA / (Sl * sm1)) * T[GS_A] - (DR / sm1) * T[GS_R] -
                      (0.5 / Sl) * (lam * DR * T[GS_DR] + mu * DA * T[GS_DA]));
        G[4] = DA * (T[GS_S0] + (c * c / (d * d)) * T[GS_SQ]);
        G[5] = DA * T[GS_N];
        G[6] = DA * (2.0 * gam * c / (d * d)) * T[GS_SQ];
        G[7] = DA * (-2.0 * K) * (T[GS_SQ] / d + d * T[GS_SQR]);
        G[8] = DA * (-2.0 * K * d * d) * T[GS_SP];
    } else {
        // S = 2: DR = D0, DA = 2 D0, mu = alpha, lambda = 2 alpha
        G[0] = 0.5 * T[GS_R] - T[GS_A];
        G[1] = D0 * (T[GS_DA] - T[GS_DR]);
        G[2] = al * D0 * (T[GS_R] - T[GS_A]);
        G[3] = 2.0 * D0 * T[GS_Z2];
        G[4] = 2.0 * D0 * T[GS_N];
        G[5] = -4.0 * D0 * x[3] * T[GS_Z1];
    }
}

template <typename S, int M, bool Full = false>
__device__ __forceinline__ void run_adjoint(const BArgs<S>& A, const Item& it, const ItemCtx& x,
                                            unsigned char* __restrict__ lds) {
    const SetDev& d = A.set;
    const int N = d.N;
    const Rec<S>* __restrict__ pbuf = reinterpret_cast<const Rec<S>*>(lds);
    Vec4<S>* __restrict__ ab =
        reinterpret_cast<Vec4<S>*>(lds + lds_param_bytes<S>(it.nc)) + (size_t)x.q * x.npad;
    Geo<S, M, Full> g;
    g.load(d, x.atom, x.active);
    constexpr int MM = M > 0 ? M : 1;
    constexpr int NL = GradSums<Full>::value;
    constexpr int NV = Full ? kNVGradTF : kNVGrad;
    double* __restrict__ red = reinterpret_cast<double*>(lds - kRedBytes);
    int jl[MM];
#pragma unroll
    for (int m = 0; m < M; ++m) jl[m] = d.jl[(size_t)m * N + x.atom];
    __syncthreads();                                   // the records
    auto flush = [&](int step) __attribute__((always_inline)) {
        const int cl = x.q + step * x.R;
        if (cl < it.nc) flush_sums<MODE_FIT, NV>(A, x, it.c0 + cl, NL, true, red);
    };

    for (int step = 0; step < x.steps; ++step) {
        const int cl = x.q + step * x.R;
        const bool group_ok = cl < it.nc;
        const int clv = group_ok ? cl : 0;
        const int c = it.c0 + clv;
        const Rec<S>& prec = pbuf[clv];
        // this atom's force residual, from the fitness call (lanes outside the
        // structure: another atom's, and f_C = 0)
        const S* r = A.resid + (size_t)c * 3 * N;
        const S ax = r[x.atom], ay = r[(size_t)N + x.atom], az = r[(size_t)2 * N + x.atom];
        ab[x.la] = Vec4<S>{ax, ay, az, S(0)};
        exchange_sync(x.block_sync);
        if (x.block_sync && step > 0) flush(step - 1);
        S L[NL];
        adjoint_sums<S, M, Full>(
            g, prec, ax, ay, az,
            [&](int m) {
                // read afresh on every use (a reused value would stay live)
                int jm = jl[m];
                asm volatile("" : "+v"(jm));
                return ab[jm];
            },
            A.coef + ((size_t)c * d.S + x.s) * 8, L);
        exchange_sync(x.block_sync);
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = k < NL ? (double)L[k < NL ? k : 0] : 0.0;
        store_group<MODE_FIT, NV>(v, A, x, group_ok, c, 0, Full ? 0xff : 0x7f, true, red);
        if constexpr (Full) {
            double u[8];
            u[0] = (double)L[8];
#pragma unroll
            for (int k = 1; k < 8; ++k) u[k] = 0.0;
            store_group<MODE_FIT, NV>(u, A, x, group_ok, c, 8, 0x01, true, red);
        }
    }
    if (x.block_sync) {
        __syncthreads();
        flush(x.steps - 1);
    }
}

template <typename S, int MC, bool Full>
__device__ __forceinline__ void adjoint_item(const BArgs<S>& A, const Item& it, unsigned char* lds) {
    const ItemCtx x = item_ctx(A.set, it);
    decode_item<S, Full>(A, it, lds);
    const int Mw = x.Mw;
    if (Mw < 0) {
        run_idle(x.block_sync ? 2 * x.steps + 1 : 0);
        return;
    }
    dispatch_m<ClassLo<MC>::value, MC>(Mw, [&](auto mv) {
        run_adjoint<S, decltype(mv)::value, Full>(A, it, x, lds);
    });
}

// The float minimal class of up to four neighbours runs four wavefronts a SIMD (128
// registers; 57 us in the gradient of 64 candidates x 300 structures at three, 47 at four).
template <typename S, int MC, bool Full = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MC <= 4 && sizeof(S) == 4 && !Full ? 4 : 1)))
void k_adjoint(BArgs<S> A) {
    extern __shared__ __align__(32) unsigned char lds_raw[];
    // without bins, block b has item b
    const int b0 = A.bin_off ? A.bin_off[blockIdx.x] : (int)blockIdx.x;
    const int b1 = A.bin_off ? A.bin_off[blockIdx.x + 1] : b0 + 1;
    for (int i = b0; i < b1; ++i) {
        const Item it = load_item(A.items + i);
        adjoint_item<S, MC, Full>(A, it, lds_raw + kRedBytes);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Large structures (more atoms than one block holds): two passes per
// candidate.  Pass 1 writes every bond gradient to global memory and the
// energy, virial and heat current partials; pass 2 gathers forces, per-atom
// virial and the force residual.
// ---------------------------------------------------------------------------
// One staged bond gradient of the two-pass path: x, y, z and an unused
// fourth value, so that the gather reads a partner's reverse bond with one
// vector load (one cache line) instead of three scattered ones.
template <typename S>
struct Stage4;
template <>
struct Stage4<float> {
    using T = float4;
};
template <>
struct Stage4<double> {
    using T = double4;
};

struct LArgs {
    int s, c0;                 // structure, first candidate of the chunk
    void* gbuf;                // [chunk][nbs] of Stage4<S> (x, y, z, unused)
    // where the blocks' partial sums go, [candidate][pslots][nv] (null: nowhere):
    // the set's slots, one per block of a structure over the batching limit, as
    // many as the site kernel has blocks (fin), or a buffer of their own that
    // k_sum_blocks adds up (a batched structure sent to the two-pass path has one slot)
    double* part;
    int pslots;
    // the structure's first atom, atom count, bond count, first partial-sum
    // slot and largest coordination, copied from the host tables so no kernel
    // waits on reading them
    int a0, ns, nbs, slot0, kmax;
    // evaluation of a set of one structure: the gather's first block adds up the
    // site kernel's sums and writes energy, virial and heat current (form: 1 for
    // Tersoff-form parameters)
    int fin, form;
    int gblock;                // with fin: threads of a gather block
};

// Store a block's sums, values off + k for the k set in mask: its wavefronts'
// group sums (lanes with (lane & 7) == 0 hold value vidx) added in wavefront
// order through LDS.  Every thread of the block calls it; a wavefront with no
// atom passes sum = 0 and vidx = (lane >> 3).
__device__ __forceinline__ void large_store(const LArgs& L, int nv, int c, double sum, int vidx, unsigned mask,
                                            int off, double (*sh)[8]) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((lane & 7) == 0) sh[w][vidx] = sum;
    __syncthreads();
    const int k = threadIdx.x;
    if (k < 8 && ((mask >> k) & 1)) {
        double t = sh[0][k];
        for (int q = 1; q < nw; ++q) t += sh[q][k];
        L.part[((size_t)c * L.pslots + L.slot0 + blockIdx.x) * nv + off + k] = t;
    }
    __syncthreads();
}

template <typename S, int M, bool E64, bool Full>
__device__ __forceinline__ void run_large_site(const BArgs<S>& A, const LArgs& L, int la, int atom,
                                               bool active, double& sum, int& vidx, double& jsum, int& jvidx,
                                               int rows = M) {
    const SetDev& d = A.set;
    const int N = d.N;
    Geo<S, M, Full, false> g;
    g.load(d, atom, active, rows);
    constexpr int MM = M > 0 ? M : 1;
    const int c = L.c0 + blockIdx.y;
    const int nbs = L.nbs;
    const int Mi = active ? d.nnb[atom] : 0;
    const int lb = active ? d.lbo[atom] : 0;
    // the bond partners' velocities (caller's numbering): read beside the
    // geometry where the registers hold them, else when they are used
    constexpr bool kEarly = M <= 6;
    int oj[MM];
    S vj[kEarly ? MM : 1][3];
    if (A.vel) {
#pragma unroll
        for (int m = 0; m < M; ++m) oj[m] = active && m < rows ? max(d.nbr_j[(size_t)m * N + atom], 0) : 0;
        if constexpr (kEarly) {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int k = 0; k < 3; ++k) vj[m][k] = (S)A.vel[(size_t)k * N + oj[m]];
        }
    }
    Rec<S> rec;
    decode_record<S, Full>(A.x + Form<Full>::nx * (size_t)c, rec);
    Cand<S, Full> p;
    load_cand(rec, p);
    double U;
    S Gx[MM], Gy[MM], Gz[MM];
    // about one wavefront per SIMD for a large structure: the bonds' float64
    // energy chains interleave
    site_eval<S, M, E64, Full, false, false>(g, p, U, Gx, Gy, Gz);
    using V4 = typename Stage4<S>::T;
    V4* gb = reinterpret_cast<V4*>(L.gbuf) + (size_t)blockIdx.y * nbs;
    if (active) {
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (m < Mi) gb[lb + m] = V4{Gx[m], Gy[m], Gz[m], S(0)};
    }
    S w6[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) w6[k] = S(0);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const S rm = g.length(m), dx = rm * g.ux[m], dy = rm * g.uy[m], dz = rm * g.uz[m];
        w6[0] -= dx * Gx[m]; w6[1] -= dy * Gy[m]; w6[2] -= dz * Gz[m];
        w6[3] -= dy * Gz[m]; w6[4] -= dz * Gx[m]; w6[5] -= dx * Gy[m];
    }
    double v[8];
    v[0] = active ? (double)U : 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) v[1 + k] = active ? (double)w6[k] : 0.0;
    v[7] = 0.0;
    sum = group_reduce8_t<64>(v, &vidx);
    if (A.vel) {
        // heat current sum_i W_i v_i, bond by bond from the centre's side: W_i
        // has -d (x) G of every bond (d, G) that ends at i
        S j3[3] = {S(0), S(0), S(0)};
#pragma unroll
        for (int m = 0; m < M; ++m) {
            S vx, vy, vz;
            if constexpr (kEarly) {
                vx = vj[m][0]; vy = vj[m][1]; vz = vj[m][2];
            } else {
                vx = (S)A.vel[oj[m]]; vy = (S)A.vel[(size_t)N + oj[m]]; vz = (S)A.vel[(size_t)2 * N + oj[m]];
            }
            const S gv = Gx[m] * vx + Gy[m] * vy + Gz[m] * vz;
            const S rm = g.length(m), dx = rm * g.ux[m], dy = rm * g.uy[m], dz = rm * g.uz[m];
            j3[0] -= dx * gv; j3[1] -= dy * gv; j3[2] -= dz * gv;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = active && k < 3 ? (double)j3[k < 3 ? k : 0] : 0.0;
        jsum = group_reduce8_t<64>(v, &jvidx);
    }
}

// E64: float64 energy terms (the float path's energy/force/virial mode).
template <typename S, int MC, bool E64, bool Full = false>
__global__ __launch_bounds__(256) void k_large_site(BArgs<S> A, LArgs L) {
    const SetDev& d = A.set;
    const int a0 = L.a0, Ns = L.ns;
    const int la = blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = la < Ns;
    const int atom = a0 + (active ? la : 0);
    __shared__ double sh[kLargeBlock / 64][8];
    double sum = 0.0, jsum = 0.0;
    int vidx = (threadIdx.x & 63) >> 3, jvidx = vidx;
    if constexpr (MC <= 4) {
        // one variant for the class: the geometry rows (up to the structure's
        // largest coordination) are read without first waiting for the
        // wavefront's bond counts
        if ((la & ~63) < Ns) run_large_site<S, MC, E64, Full>(A, L, la, atom, active, sum, vidx, jsum, jvidx, L.kmax);
    } else {
        // the wavefront's first atom has its largest coordination (sorted)
        const int first = __builtin_amdgcn_readfirstlane(la & ~63);
        const int Mw = first < Ns ? d.nnb[a0 + first] : -1;
        if (Mw >= 0)
            dispatch_m<ClassLo<MC>::value, MC>(Mw, [&](auto mv) {
                run_large_site<S, decltype(mv)::value, E64, Full>(A, L, la, atom, active, sum, vidx, jsum, jvidx);
            });
    }
    // no partial sums when only the staged bond gradients are wanted
    if (L.part) large_store(L, A.nv, L.c0 + blockIdx.y, sum, vidx, 0x7f, 0, sh);
    if (L.part && A.vel) large_store(L, A.nv, L.c0 + blockIdx.y, jsum, jvidx, 0x07, 8, sh);
}

// Energy, virial and heat current of candidate c from the site kernel's sums,
// one block of any number of wavefronts: consecutive threads on consecutive
// values (thread t only ever sees value t % 16), sixteen loads in flight each,
// then the lanes of equal value and the wavefronts in order.
template <typename S>
__device__ __forceinline__ void finish_eval(const BArgs<S>& A, const LArgs& L, int c, double (*sh)[16]) {
    static_assert(kNVEval == 16, "sixteen values per slot");
    const double* base = L.part + (size_t)c * L.pslots * kNVEval;
    const int total = L.pslots * kNVEval, nt = blockDim.x;
    double acc = 0.0;
    for (int e = threadIdx.x; e < total; e += 16 * nt) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = e + u * nt < total ? base[e + u * nt] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
    }
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    const int lane = threadIdx.x & 63, k = threadIdx.x;
    if (lane < 16) sh[threadIdx.x >> 6][lane] = acc;
    __syncthreads();
    if (k >= 11 || k == 7) return;
    double t = sh[0][k];
    for (int w = 1; w < nt >> 6; ++w) t += sh[w][k];
    const bool ok = L.form ? params_valid<true>(A.x + 9 * (size_t)c) : params_valid<false>(A.x + 6 * (size_t)c);
    if (!ok) t = __longlong_as_double(0x7ff8000000000000ll);
    if (k == 0) { if (A.energy) A.energy[c] = t; }
    else if (k <= 6) { if (A.virial) A.virial[(size_t)c * 6 + k - 1] = t; }
    else if (A.heat) A.heat[(size_t)c * 3 + k - 8] = t;
}

// Bound by memory latency and, for a large cell, by its 40 MB a call through the
// caches: the rows of four bonds are read together, predicated, so that the
// round trips go with the quads of the structure's coordination (8,000 atoms with
// skin neighbours 11.0 us bond by bond, 10.0 us).  For a set of one structure a
// block before the atoms' finishes the sums meanwhile: its own launch took 4.3 us
// of a 23.3 us call (64,000 atoms, float64), 20.6 us without.
template <typename S, int MODE, int MC>
__global__ __launch_bounds__(256) void k_large_gather(BArgs<S> A, LArgs L) {
    const SetDev& d = A.set;
    const int N = d.N;
    const int a0 = L.a0, Ns = L.ns;
    const int nbs = L.nbs;
    const int c = L.c0 + blockIdx.y;
    if constexpr (MODE == MODE_EVAL) {
        __shared__ double shf[kLargeBlock / 64][16];
        if (L.fin && blockIdx.x == 0) {
            finish_eval(A, L, c, shf);
            return;
        }
    }
    const int la = (blockIdx.x - (MODE == MODE_EVAL && L.fin)) * blockDim.x + threadIdx.x;
    const bool active = la < Ns;
    const int atom = a0 + (active ? la : 0);
    using V4 = typename Stage4<S>::T;
    const V4* gb = reinterpret_cast<const V4*>(L.gbuf) + (size_t)blockIdx.y * nbs;
    const GeomArrays<S> G = geom_of<S>(d);
    // The reverse-bond indices (rows up to the structure's largest
    // coordination) are read in the same memory round trip as the atom's
    // bond count; the staged gradients of its bonds in the next.
    const int rows = L.kmax < MC ? L.kmax : MC;
    int rv[MC];
#pragma unroll
    for (int m = 0; m < MC; ++m) rv[m] = active && m < rows ? d.revc[(size_t)m * N + atom] : 0;
    const int Mi = active ? d.nnb[atom] : 0, lb = active ? d.lbo[atom] : 0;
    S Fx = S(0), Fy = S(0), Fz = S(0);
    S wi[9];
    for (int k = 0; k < 9; ++k) wi[k] = S(0);
#pragma unroll
    for (int m0 = 0; m0 < MC; m0 += 4) {
        if (m0 >= rows) break;
        V4 rg[4], og[4];
        S dx[4], dy[4], dz[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m = m0 + q;
            const bool ok = m < Mi;
            rg[q] = ok ? gb[rv[m]] : V4{S(0), S(0), S(0), S(0)};
            og[q] = ok ? gb[lb + m] : V4{S(0), S(0), S(0), S(0)};
            if (MODE == MODE_EVAL) {
                const size_t o = (size_t)m * N + atom;
                if constexpr (sizeof(S) == 4) {
                    const float4 u = ok ? G.pk0[o] : make_float4(0.f, 0.f, 0.f, 0.f);
                    dx[q] = u.w * u.x; dy[q] = u.w * u.y; dz[q] = u.w * u.z;
                } else {
                    const S rr = ok ? G.rhi[o] : S(0), ux = ok ? G.ux[o] : S(0), uy = ok ? G.uy[o] : S(0),
                            uz = ok ? G.uz[o] : S(0);
                    dx[q] = rr * ux; dy[q] = rr * uy; dz[q] = rr * uz;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const S rx = rg[q].x, ry = rg[q].y, rz = rg[q].z;
            Fx += og[q].x - rx;
            Fy += og[q].y - ry;
            Fz += og[q].z - rz;
            if (MODE == MODE_EVAL) {
                wi[0] += dx[q] * rx; wi[1] += dx[q] * ry; wi[2] += dx[q] * rz;
                wi[3] += dy[q] * rx; wi[4] += dy[q] * ry; wi[5] += dy[q] * rz;
                wi[6] += dz[q] * rx; wi[7] += dz[q] * ry; wi[8] += dz[q] * rz;
            }
        }
    }
    if (MODE == MODE_FIT) {
        __shared__ double sh[kLargeBlock / 64][8];
        double v[8];
        for (int k = 0; k < 8; ++k) v[k] = 0.0;
        int vidx;
        const S* fr = fref_of<S>(d);
        if (active) {
            const S ax = Fx - fr[atom], ay = Fy - fr[(size_t)N + atom], az = Fz - fr[(size_t)2 * N + atom];
            v[7] = (double)(ax * ax + ay * ay + az * az);
        }
        const double sum = group_reduce8_t<64>(v, &vidx);
        large_store(L, A.nv, c, sum, vidx, 0x80, 0, sh);
    } else if (active) {
        const int orig = d.perm[atom];
        if (A.force) {
            double* f = A.force + (size_t)c * 3 * N;
            f[orig] = (double)Fx; f[(size_t)N + orig] = (double)Fy; f[(size_t)2 * N + orig] = (double)Fz;
        }
        if (A.atom_virial) {
            double* w = A.atom_virial + (size_t)c * 9 * N;
            for (int k = 0; k < 9; ++k) w[(size_t)k * N + orig] = (double)wi[k];
        }
    }
}

// ---------------------------------------------------------------------------
// Fitness gradient of the two-pass structures.  k_large_site stages the bond
// gradients of a candidate chunk (as for the fitness), k_large_residual turns
// them into the force residuals a_i = F_i - F*_i, staged [chunk][3][Ns], and
// k_large_adjoint forms every atom's grad sums (adjoint_sums) with the
// residuals of its bond partners read from there; its partial sums go to one
// slot per 256-atom block (a structure of at most 512 atoms: to its one slot by
// k_sum_blocks).
// ---------------------------------------------------------------------------
template <typename S>
__global__ __launch_bounds__(256) void k_large_residual(BArgs<S> A, LArgs L, S* __restrict__ abuf) {
    const SetDev& d = A.set;
    const int N = d.N;
    const int a0 = L.a0, Ns = L.ns;
    const int nbs = L.nbs;
    const int la = blockIdx.x * blockDim.x + threadIdx.x;
    if (la >= Ns) return;
    const int atom = a0 + la;
    using V4 = typename Stage4<S>::T;
    const V4* gb = reinterpret_cast<const V4*>(L.gbuf) + (size_t)blockIdx.y * nbs;
    S Fx = S(0), Fy = S(0), Fz = S(0);
    const int Mi = d.nnb[atom], lb = d.lbo[atom];
    for (int m = 0; m < Mi; ++m) {
        const int r = d.revc[(size_t)m * N + atom];
        const V4 rg = gb[r], og = gb[lb + m];
        Fx += og.x - rg.x;
        Fy += og.y - rg.y;
        Fz += og.z - rg.z;
    }
    const S* fr = fref_of<S>(d);
    S* a = abuf + (size_t)blockIdx.y * 3 * Ns;
    a[la] = Fx - fr[atom];
    a[Ns + la] = Fy - fr[(size_t)N + atom];
    a[2 * Ns + la] = Fz - fr[(size_t)2 * N + atom];
}

template <typename S, int M, bool Full>
__device__ __forceinline__ void run_large_adjoint(const BArgs<S>& A, const LArgs& L, int la, int atom,
                                                  bool active, int Ns, const S* __restrict__ abuf,
                                                  double& sum, int& vidx, double& sum2, int& vidx2) {
    const SetDev& d = A.set;
    const int N = d.N;
    constexpr int MM = M > 0 ? M : 1;
    constexpr int NL = GradSums<Full>::value;
    Geo<S, M, Full> g;
    g.load(d, atom, active, d.kcap);
    int jl[MM];
#pragma unroll
    for (int m = 0; m < M; ++m) jl[m] = m < d.kcap ? d.jl[(size_t)m * N + atom] : 0;
    const int c = L.c0 + blockIdx.y;
    Rec<S> rec;
    decode_record<S, Full>(A.x + Form<Full>::nx * (size_t)c, rec);
    const S* a = abuf + (size_t)blockIdx.y * 3 * Ns;
    const int own = atom - L.a0;
    const S ax = a[own], ay = a[Ns + own], az = a[2 * Ns + own];
    S sums[NL];
    // lanes past the structure have f_C = 0 on every bond: every sum is zero
    adjoint_sums<S, M, Full>(
        g, rec, ax, ay, az,
        [&](int m) {
            int jm = jl[m];
            asm volatile("" : "+v"(jm));
            return Vec4<S>{a[jm], a[Ns + jm], a[2 * Ns + jm], S(0)};
        },
        A.coef + ((size_t)c * d.S + L.s) * 8, sums);
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = k < NL ? (double)sums[k < NL ? k : 0] : 0.0;
    sum = group_reduce8(v, 64, &vidx);
    if constexpr (Full) {
        double u[8];
        u[0] = (double)sums[8];
#pragma unroll
        for (int k = 1; k < 8; ++k) u[k] = 0.0;
        sum2 = group_reduce8(u, 64, &vidx2);
    }
}

// Variant that a wavefront of largest coordination Mw runs in the class above 4;
// rows past its coordination are padding bonds.  A variant whose pair sums come
// from moments reads the table that exists only for sets above kPairMax
// neighbours, so it may serve such wavefronts only.
template <typename S, bool Full>
constexpr int large_adjoint_m(int Mw) {
    return Geo<S, 8, Full>::kMoments && Mw <= kPairMax ? kPairMax : Mw <= 8 ? 8 : kMaxNbr;
}
template <typename S, bool Full>
constexpr bool large_adjoint_tables_exist() {
    for (int Mw = 0; Mw <= kMaxNbr; ++Mw) {
        const int m = large_adjoint_m<S, Full>(Mw);
        const bool moments = m == kMaxNbr ? Geo<S, kMaxNbr, Full>::kMoments
                             : m == 8     ? Geo<S, 8, Full>::kMoments
                                          : Geo<S, kPairMax, Full>::kMoments;
        if (m < Mw || (moments && Mw <= kPairMax)) return false;
    }
    return true;
}

template <typename S, int MC, bool Full>
__global__ __launch_bounds__(256) void k_large_adjoint(BArgs<S> A, LArgs L, const S* __restrict__ abuf) {
    const SetDev& d = A.set;
    const int a0 = L.a0, Ns = L.ns;
    const int la = blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = la < Ns;
    const int atom = a0 + (active ? la : 0);
    const int first = __builtin_amdgcn_readfirstlane(la & ~63);
    const int Mw = first < Ns ? d.nnb[a0 + first] : -1;
    __shared__ double sh[kLargeBlock / 64][8];
    double sum = 0.0, sum2 = 0.0;
    int vidx = (threadIdx.x & 63) >> 3, vidx2 = vidx;
    auto run = [&](auto mv) {
        run_large_adjoint<S, decltype(mv)::value, Full>(A, L, la, atom, active, Ns, abuf, sum, vidx, sum2, vidx2);
    };
    if (Mw >= 0) {                              // a wavefront with no atom adds zeros
        if constexpr (MC <= 4) {
            dispatch_m<0, MC>(Mw, run);
        } else {
            static_assert(MC == kMaxNbr && large_adjoint_tables_exist<S, Full>(), "see large_adjoint_m");
            const int m = large_adjoint_m<S, Full>(Mw);
            if (m == kMaxNbr) run(std::integral_constant<int, kMaxNbr>{});
            else if (m == 8) run(std::integral_constant<int, 8>{});
            else if constexpr (large_adjoint_m<S, Full>(0) == kPairMax) run(std::integral_constant<int, kPairMax>{});
        }
    }
    const int c = L.c0 + blockIdx.y;
    large_store(L, A.nv, c, sum, vidx, Full ? 0xffu : 0x7fu, 0, sh);
    if constexpr (Full) large_store(L, A.nv, c, sum2, vidx2, 0x01, 8, sh);
}

// Launchers, one per kernel family (defined in the mt_k_*.hip units).
hipError_t launch_fit32(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_eval32(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_fit64(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_eval64(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_adj32(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_adj64(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_adj32f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                         hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_adj64f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                         hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// The fitness kernels that also write the force residuals (A.resid), for the
// gradient's fitness call; the launch_fit* launchers pick them when A.resid
// is set.
hipError_t launch_fitr32(int mc, int full, dim3 g, dim3 b, size_t lds, hipStream_t st,
                         const BArgs<float>& A, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_fitr64(int mc, int full, dim3 g, dim3 b, size_t lds, hipStream_t st,
                         const BArgs<double>& A, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_fitr32f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                          hipEvent_t e0, hipEvent_t e1);
// Tersoff-form (nine-parameter) batched families.
hipError_t launch_fit32f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                         hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_eval32f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A,
                          hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_fit64f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                         hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_eval64f(int mc, dim3 g, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A,
                          hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// Plain-schedule launchers (one block, one item); mode is MODE_FIT or MODE_EVAL,
// full selects the Tersoff form.
hipError_t launch_plain32(int mode, bool full, int mc, dim3 b, size_t lds, hipStream_t st,
                          const BArgs<float>& A);
hipError_t launch_plain64(int mode, bool full, int mc, dim3 b, size_t lds, hipStream_t st,
                          const BArgs<double>& A);
hipError_t launch_plain32f(int mode, int mc, dim3 b, size_t lds, hipStream_t st, const BArgs<float>& A);
hipError_t launch_plain64f(int mode, int mc, dim3 b, size_t lds, hipStream_t st, const BArgs<double>& A);
hipError_t launch_large32(int mc, int mode, int full, dim3 g, dim3 b, hipStream_t st,
                          const BArgs<float>& A, const LArgs& L);
hipError_t launch_large64(int mc, int mode, int full, dim3 g, dim3 b, hipStream_t st,
                          const BArgs<double>& A, const LArgs& L);
// Two-pass fitness gradient of one structure and candidate chunk: force
// residuals into abuf from the bond gradients staged by launch_large* in
// MODE_STAGE, then the grad sums.
hipError_t launch_large_adj32(int mc, int full, dim3 g, dim3 b, hipStream_t st, const BArgs<float>& Afit,
                              const BArgs<float>& Aadj, const LArgs& L, float* abuf);
hipError_t launch_large_adj64(int mc, int full, dim3 g, dim3 b, hipStream_t st, const BArgs<double>& Afit,
                              const BArgs<double>& Aadj, const LArgs& L, double* abuf);
// The Tersoff form's residual and grad-sum kernels of the two-pass gradient.
hipError_t launch_large_adj32f(int mc, dim3 g, dim3 b, hipStream_t st, const BArgs<float>& A,
                               const LArgs& L, float* abuf);
hipError_t launch_large_adj64f(int mc, dim3 g, dim3 b, hipStream_t st, const BArgs<double>& A,
                               const LArgs& L, double* abuf);

}  // namespace mt

// Internal declarations shared by the HIP translation units of the library.
//
// Data layout in HBM (all "sorted" atom indices: inside each structure the atoms
// are reordered by descending coordination number, so that the atoms of one
// wavefront have nearly the same number of neighbours; `perm` maps back to the
// caller's numbering):
//
//   per structure s : st_off[s]     first sorted atom, st_off[S] = N
//                     st_boff[s]    first bond (CSR over sorted atoms)
//                     st_npad[s]    atoms rounded up to 8/16/32/64 or a multiple of 64
//                     st_kmax[s]    largest coordination in s
//                     st_slot[s]    first partial-sum slot of s
//   per atom a      : perm[a], nnb[a] (coordination), lbo[a] (first bond of a,
//                     relative to st_boff[s]), xbase[a] (exchange slot, below)
//   per bond slot   : slot-major arrays [m][N] (m < kcap) of float and double
//                     geometry: unit vector, length (float: hi+lo split), 1/r,
//                     f_C(r), f_C'(r)/2; int: exchange slot and CSR index of the
//                     reverse bond, neighbour atom (structure-local sorted index).
//
// Exchange slots (LDS of the batched kernels).  A replica of structure s is cut
// into chunks of G = min(npad, 64) lanes; chunk c reserves K_c * G slots, K_c
// being the largest coordination in the chunk (at least 3, the lowest variant of
// the classes above 4), and bond m of the atom in lane l of the chunk uses
// slot off_c + m * G + l.  Padded bonds (m >= coordination) own a slot too and
// their reverse index is that slot, so the exchange needs no predicates.
//
// Geometry is candidate independent (R1, R2 are fixed, not fitted), so it is
// built once per structure set and reused by every candidate.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "mt_math.h"

namespace mt {

constexpr int kMaxNbr = 16;        // template limit on coordination
constexpr int kMaxBatched = 512;   // largest structure of the batched kernel
// LDS in front of a batched block's records: the sums of up to eight wavefronts,
// sixteen values each.
constexpr int kRedBytes = 8 * 16 * 8;
// Threads per block of the two-pass kernels (evaluations of one structure of few
// atoms: see site_block); a structure over the batching limit has one partial-sum
// slot per such block.
constexpr int kLargeBlock = 256;
constexpr int kNVFit = 8;          // partial sums per slot: E, W6, |F - F*|^2
constexpr int kNVEval = 16;        // E, W6, |F-F*|^2, J3, unused
// Sums behind dZ/dx (see GradSum in mt_kernels.h): seven, one unused; the
// Tersoff form's nine, seven unused.
constexpr int kNVGrad = 8;
constexpr int kNVGradTF = 16;

// Decoded parameter record, filled per work item in LDS.  Both potential forms
// share it: f_R = DR e^{-lambda (r - r0)}, f_A = DA e^{-mu (r - r0)} with
// lambda = alpha sqrt(2S), mu = alpha sqrt(2/S), DR = D0/(S-1), DA = S D0/(S-1)
// (Sec. II.B Eqs. 11-14; S = 2 in the minimal potential); zeta = ZS sum_k f_C g(theta)
// with g = (cos - h)^2 and ZS = beta (minimal), or g = g^T = gamma + K t^2 / (d^2 + t^2),
// t = cos - h, K = gamma c^2 / d^2 and ZS = 1 (Tersoff form, Sec. II.A Eq. 8).
// The float path's energy terms are evaluated in float64: their parameters stand
// here in float64 too, so that no lane converts or joins them per candidate.
template <typename S>
struct alignas(16) Rec {
    double aA64, r0, DR64, ninv2n64;   // mu log2(e), r0, DR, -1/(2n)
    double aR64, DA64;                 // lambda log2(e), DA (Tersoff form)
    S aA, DR, DA, n, ninv2n;
    S h, hlo;                          // hlo: h - h_S (zero in double records)
    S zs, hmu, ccs;                    // zeta scale; mu / 2; gradient scale: beta / 2, or 1 / 2
    S valid;                           // 1 if the candidate is inside the potential's domain
    S aR, hlambda;                     // lambda log2(e), lambda / 2 (Tersoff form, with the next four)
    S gam, K, d2, Kd2;                 // gamma, gamma c^2 / d^2, d^2, K d^2
};

// One (structure, candidate range) work item of the batched kernels, with the
// structure's own numbers: a block learns all of them in one load.
struct Item {
    int s;
    int c0;
    int nc;
    int cost;       // relative cost used for scheduling
    int a0, ns;     // the structure's first atom and atom count
    int npad;
    int slot;       // its first partial-sum slot
    int xsz;        // exchange slots of one replica
    int R;          // replicas a block holds
    int unused[2];  // 48 bytes
};

template <typename S>
struct GeomArrays {
    const S* ux; const S* uy; const S* uz;
    const S* rhi; const S* rlo; const S* rinv;
    const S* fc; const S* hfcp;     // f_C and f_C'/2
    // float only: the same geometry packed per bond slot as two 4-vectors,
    // (ux, uy, uz, r_hi) and (r_lo, 1/r, f_C, f_C'/2), [kcap][N] each.  The float
    // kernels read these two alone; without the unpacked arrays the other buffers
    // lie elsewhere and the 64,000-atom force call is slower (float64 21.1 -> 21.7
    // us, float 17.1 -> 17.4)
    const float4* pk0; const float4* pk1;
};

struct SetDev {
    int S, N, kcap, nb, nslots;
    const int* st_off; const int* st_boff;
    const int* st_slot;
    const int* perm; const int* nnb; const int* lbo;
    const int* xbase;                           // [N] first exchange slot of the atom
    const int* rev;                             // [kcap][N] exchange slot of the reverse bond
    const int* revc;                            // [kcap][N] structure-local CSR index of it
    const int* jl;                              // [kcap][N] structure-local neighbour atom
    const int* nbr_j;                           // [kcap][N] neighbour atom, caller's numbering (-1: padding)
    GeomArrays<float> gf;
    GeomArrays<double> gd;
    // [15][N] cos(theta_jk) of the bond pairs j < k < 6, pair k (k - 1) / 2 + j:
    // float64 unit-vector products rounded once (zero for padding bonds)
    const float* gcs;
    // angular moments (S, H, V) of every bond over the atom's other bonds, for
    // sets with more than kPairMax neighbours somewhere (null otherwise):
    // [kcap][N] float4 (fourth unused)
    const float4* gam;
    const float* fref32;  const double* fref64; // [3][N] sorted order
};

// Largest coordination whose angular sums run over bond pairs in the float
// minimal form; above it they come from moments.  About 52 operations a bond by moments
// against 13 a pair (20 uncached, M > 6): equal between 6 and 7 neighbours.
constexpr int kPairMax = 6;

// Pairs of bonds whose cos(theta) the pair table holds (bonds 0-5).
constexpr int kCosPairs = 15;

// ---------------------------------------------------------------------------
// Host-side helpers shared by the translation units.
// ---------------------------------------------------------------------------
void set_error(const std::string& msg);
int hip_fail(hipError_t e, const char* what);

}  // namespace mt

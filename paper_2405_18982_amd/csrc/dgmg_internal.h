// Internal declarations shared by the host orchestration (dgmg_api.cpp) and
// the per-(dimension, degree) kernel translation units (dgmg_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dgmg {

constexpr int kMaxDegree = 7;
constexpr int kMaxLevels = 21;   // levels 0..20 (finest level L <= 20)
// workgroup shapes of apply: 0, 1 patches per workgroup; 2 face data in
// registers; 3 several right-hand sides of one patch per workgroup
constexpr int kApplyShapes = 4;
// workgroup shapes of the smoother: 0..7 patches per workgroup x prefetch of
// b x (two waves per patch | one patch per workgroup); 8..11 several
// right-hand sides of one patch per workgroup (two slot counts) x prefetch
constexpr int kSmoothShapes = 12;

// Where the Dirichlet smoothers take the direct form (one solve for the new
// values) and not a residual by operator passes.  On the shortest lines its
// face passes outweigh the operator passes they replace: a smoothing step of
// 3-D Q1 takes 33.1 us on 8^3 cells and 105.6 us on 64^3 by operator passes, 36.7
// and 109.4 us directly; 2-D Q2 on 8^2 cells 16.4 against 17.6 us, 2-D Q3 on 64^2
// (three right-hand sides) 21.3 both, 2-D Q7 on 128^2 53.0 against 40.3 us.
constexpr bool direct_smoother(int dim, int k) { return dim == 3 ? k >= 2 : k >= 4; }
// Only levels with fewer cells a direction than this do.  In 2-D the direct form
// reads and writes lines along y, a cell row in FP32 20 to 28 bytes for Q4..Q6, where
// the residual form has x-lines; that costs nothing while a level sits in the
// caches and few patches wait on their phases, and up to a third where it is bound by
// memory.  FP32 smoothing steps, direct / residual form: Q4 64^2 cells 21.1 / 21.1 us, 256^2
// 37.8 / 35.3, 512^2 94.7 / 81.2; Q5 128^2 27.4 / 29.8, 256^2 48.8 / 47.8, 512^2 117.6 / 105.9;
// Q6 64^2 25.7 / 26.9, 128^2 31.8 / 31.9 (with 16 right-hand sides 171 / 144), 256^2 61.3 /
// 56.1, 1024^2 822 / 626; Q7, whose rows are whole 32 bytes, 128^2 33.1 / 36.6, 512^2 163 /
// 164.  FP64 and 3-D: direct everywhere.
constexpr int kAllLevels = 1 << 30;
constexpr int direct_below(int dim, int k, int bytes) {
  return dim == 2 && bytes == 4 && k >= 4 && k <= 6 ? (k == 5 ? 256 : 128) : kAllLevels;
}

// Reference (h = 1, kappa = 1) data of Q_K on a two-cell patch that depends
// on the penalty, in the arithmetic type T of the kernels that read them.
// Built on the host in FP64 (setup.cpp) and uploaded once per context.  (The
// basis matrices that depend on K alone -- mass, stiffness, end derivatives,
// prolongation -- are compile-time constants, dgmg_ref1d.h.)
//   sigma : penalty factor (gamma_F = sigma / h)
//   S[t], lam[t] : fast-diagonalisation eigenpairs of patch type t on the
//         Dirichlet local space, padded to E (unused eigenvalue slots hold a
//         huge finite value)
//   MS[t], gp[t], gt[t], gm[t] : S^T M and the couplings of the Dirichlet space
//         to the dropped end nodes and the outer traces in the eigenbasis
//         (dgmg_setup.h)
//   Sf[t], lamf[t] : the same on the whole patch (Full kernel)
//   Sc[t], lamc[t] : C S on the clamped space with basis C (clamped kernel)
//   rs[s][c] : the inverse eigenvalue sums of the fast-diagonalisation solve
//         of local space s (0 Dirichlet, 1 whole patch, 2 clamped) for the
//         patch-type combination c = (tx 4 + ty) 4 + tz (2-D: tx 4 + ty),
//         computed in FP64 and rounded; 0 where a slot is unused:
//         rs[s][c][(qz E + qx) E + qy], in 2-D rs[s][c][qy E + qx].
//         s = 0 with the direct smoother, for lanes that hold x-lines:
//         rs[0][c][qx E^2 + l] of the x-line (qy, qz) of lane l, the lanes
//         running through the plane cell by cell (qy = (l' mod 2) n + i mod n,
//         qz = (l' div 2) n + i div n with l' = l div n^2, i = l mod n^2); in
//         2-D rs[0][c][qx E + qy], and the other order in rs[0][16 + c].
template <int K, typename T>
struct Tab {
  static constexpr int n = K + 1;
  static constexpr int E = 2 * n;
  T sigma;
  T S[4][E * E];
  T lam[4][E];
  T MS[4][E * E];
  T gp[4][E];
  T gt[4][E];
  T gm[4][E];
  T Sf[4][E * E];
  T lamf[4][E];
  T Sc[4][E * E];
  T lamc[4][E];
  T rs[3][64][E * E * E];
};

// The patches of one launch: patch m = (m_0, .., m_{D-1}), m_i < cnt[i], has
// its lower-left cell at lo_i = off[i] + 2 m_i and covers cells lo_i, lo_i + 1.
// The Full smoother's launches also carry the partial patches that complete
// the tiling of the mesh (off = -1: lo_i = -1 or N - 1, one cell inside).
struct PatchGrid {
  int N;       // cells per direction on the level
  int cnt[3];  // patches per direction
  int off[3];  // -1, 0 or 1
  int npatch;  // product of cnt
  int xcd_remap;  // 1: give each XCD a contiguous range of patches
  int nrhs;    // right-hand sides of the launch (set by the launchers)
  // Which patches of the direct smoother look for non-finite old values: 0 none,
  // 1 those at the domain boundary, 2 all.  A patch that found one gives none but
  // NaNs, and every later patch that shares a cell with it reads some of these
  // in its dropped layers, so a cell need be looked at only by the first patch of a
  // step that holds it: ascending from colour 0, which holds every cell, that is
  // colour 0 alone; descending, the last colour holds all cells but the
  // outermost ones, which only patches at the boundary reach.  A smoothing step
  // with every patch of every colour looking was 4% slower (3-D Q4 32^3 x 16 FP32 1592 /
  // 1533 us, Q5 16^3 FP64 96.9 / 93.3 us without), this way it is 0.5%; launches
  // without any take kernels of their own (a V-cycle of Q7 64^3 FP32 would be 1.3% slower
  // on one kernel for both).
  int guard;
  // multipliers of the divisions by cnt[0], cnt[1] (grid_magic; 0: divide)
  unsigned mul[2];
};

// r / cnt = (r * mul) >> 32 with mul = ceil(2^32 / cnt), exact while
// r (mul cnt - 2^32) < 2^32, hence for r < npatch if npatch cnt <= 2^32.  A
// true division by a launch argument is a chain of some forty instructions
// at the start of every patch.
inline void grid_magic(PatchGrid& g) {
  for (int i = 0; i < 2; ++i) {
    const bool ok = g.cnt[i] > 1 && (unsigned long long)g.npatch * (unsigned)g.cnt[i] <= (1ull << 32);
    g.mul[i] = ok ? (unsigned)(((1ull << 32) + (unsigned)g.cnt[i] - 1) / (unsigned)g.cnt[i]) : 0u;
  }
}

// Host-visible launchers of one (D, K) instantiation.  All vectors are
// [nrhs][ndof] device arrays; `tab` points to a device Tab<K, T>.
template <typename T>
struct KernelSet {
  // apply and smooth come in several tuned shapes (patches per workgroup; for
  // the smoother also whether b is prefetched)
  hipError_t (*apply[kApplyShapes])(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                         long long ndof, hipStream_t s);
  // 1 where bit 0 of the shapes (more patches per workgroup) changes anything
  int two_counts;
  // 1 where apply shape 2 (face data in registers) differs from shape 0
  int apply_rf;
  // 1 where the right-hand-side-packed apply (shape 3) holds more than one slot
  // per workgroup; slots of the packed smoother (shapes 9, 11) by variant
  int apply_rpack;
  int smooth_rpack[4];
  hipError_t (*mass)(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                     long long ndof, hipStream_t s);
  // variant: DGMG_SMOOTH_* of the context.  The Dirichlet kernels update x in
  // place (xin is ignored); the Full kernel reads xin and writes xout.  zero:
  // colour 0 of a step that starts from x = 0 (x is not read, every node of
  // xout is written).
  hipError_t (*smooth[kSmoothShapes])(const void* tab, PatchGrid g, T scale, T inv_scale, int variant,
                          int zero, const T* xin, T* xout, const T* b, int nrhs, long long ndof,
                          hipStream_t s);
  // 1 where smoother shapes 4..7 are one patch per workgroup (patches share a
  // wave otherwise), or two waves per patch (not the Full kernel); else they are
  // 0..3 again
  int one_patch;
  int smooth_split;
  // levels with fewer cells a direction take the direct form of the Dirichlet
  // smoothers, which has no prefetch shapes (0: none)
  int direct_below;
  hipError_t (*restrict_residual)(const void* tab, PatchGrid g, T scale, const T* x, const T* b,
                                  T* bc, int nrhs, long long ndof, long long ndof_c,
                                  hipStream_t s);
  hipError_t (*prolongate_add)(const void* tab, PatchGrid g, const T* xc, T* x, int nrhs,
                               long long ndof, long long ndof_c, hipStream_t s);
  hipError_t (*coarse)(const void* tab, T inv_scale, const T* b, T* x, int nrhs,
                       long long ndof, hipStream_t s);
  // levels 1 and 0 of the V-cycle in one launch (pre-smoothing from zero,
  // restriction, coarse solve, prolongation, post-smoothing); null where the
  // level-1 patches of a colour do not fit one workgroup
  // (split: two waves per patch in the smoothing stages, where bottom_split)
  hipError_t (*bottom)(const void* tab, int variant, int split, T scale1, T inv_scale1, T inv_scale0,
                       T* x1, const T* b1, T* b0, T* x0, int nrhs, long long ndof1, long long ndof0,
                       hipStream_t s);
  int bottom_split;
  // 2-D: levels 2, 1 and 0 in one launch (null where they do not fit)
  hipError_t (*bottom3)(const void* tab, int variant, T scale2, T inv_scale2, T scale1, T inv_scale1,
                        T inv_scale0, T* x2, const T* b2, T* x1, T* b1, T* b0, T* x0, int nrhs,
                        long long ndof2, long long ndof1, long long ndof0, hipStream_t s);
};

// Registration entry of one kernel translation unit.
struct KernelEntry {
  int dim;
  int degree;
  KernelSet<double> f64;
  KernelSet<float> f32;
};

}  // namespace dgmg

// Each kernel TU defines dgmg_kernels_d<D>_k<K>(KernelEntry*).
#define DGMG_KERNEL_ENTRY_NAME(D, K) dgmg_kernels_d##D##_k##K
#define DGMG_DECLARE_ENTRY(D, K) \
  extern "C" void DGMG_KERNEL_ENTRY_NAME(D, K)(dgmg::KernelEntry * e);

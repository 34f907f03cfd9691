// Patch-tile kernels of the SIPG multigrid hot path for one (dimension D,
// degree K) pair, selected by -DDGMG_D=<2|3> -DDGMG_K=<1..7>; the build
// compiles this file once per pair.
//
// Every kernel works on "patches": the 2^D cells with coordinates lo_i and
// lo_i + 1 in each direction i.  A patch carries E = 2(K+1) nodes per
// direction (patch-local index p = n c + a for cell c in {0,1}, node a).  A
// workgroup owns PPB patches, TPP = E^(D-1) threads each (one wave per patch
// for 3-D K <= 3, several 2-D patches per wave).  Work proceeds in phases
// separated by barriers; in a phase along direction `dir` each thread owns one
// 1-D line of the patch (all other coordinates fixed), contracts it in
// registers with the 1-D matrices (wave-uniform operands read through scalar
// loads from the Tab struct) and hands the result to the next phase through
// LDS.  Operator phases start along x and read their lines straight from global
// memory: an x-line of a patch is two contiguous cell rows, and its outside
// neighbours across the x-faces are the adjacent rows, so x itself never passes
// through LDS.  Smoothers by operator passes keep that x-line in registers and
// finish with another x-phase that writes x + delta back as contiguous rows; the
// direct smoothers (gs_body) start from b and end with the new values along the
// last direction, as the 3-D operator, the restriction and most prolongations end.
//
// Operator (Sec. 2.2): on a Cartesian mesh A = sum_i (x)(M .. L_i .. M), with
// reference matrices (h = 1) and A_h = kappa h^(D-2) A_ref.  The 1-D SIPG
// operator restricted to the patch is applied per cell block (Lc: both faces
// interior) plus rank-2 face terms e alpha + d beta:
//   interior face, neighbour on the left  (its x=1 side, trace t, derivative g):
//       alpha = g/2 - sigma t, beta = -t/2   on the rows e0, d0
//   interior face, neighbour on the right (its x=0 side):
//       alpha = -sigma t - g/2, beta = t/2   on the rows e1, d1
//   domain-boundary face (Nitsche), from the cell's own line v:
//       x=0: alpha = (d0.v)/2, beta = v_0/2;  x=1: alpha = -(d1.v)/2, beta = -v_k/2
// Face data of interior neighbours across y- and z-faces ("ext") is gathered
// per face node into LDS and contracted with the tangential masses on the fly,
// giving the sum-factorised order
//   a = M_x x, b = L_x x;  c = M_y b + L_y a, d = M_y a;  y = M_z c + L_z d.
#include "dgmg_internal.h"
#include "dgmg_ref1d.h"

#ifndef DGMG_D
#error "DGMG_D must be defined"
#endif
#ifndef DGMG_K
#error "DGMG_K must be defined"
#endif

// Multiply-adds are fused only within one expression (never across
// statements), so every kernel variant that writes an output with the same
// expressions -- one or two waves per patch, fused or separate launches --
// computes it bit for bit alike, whatever the surrounding control flow.
#pragma clang fp contract(on)

namespace dgmg {
namespace {

constexpr int D = DGMG_D;
constexpr int K = DGMG_K;
constexpr int n = K + 1;
constexpr int E = 2 * n;
constexpr int NL = (D == 2) ? E : E * E;            // lines per direction
constexpr int NC = (D == 2) ? n * n : n * n * n;    // nodes per cell
constexpr int NCP = (D == 2) ? 4 : 8;               // cells per patch
constexpr int SY = E + 1;                           // padded LDS strides
// 8 more for 8-node cells: with the lanes cell by cell (8 x 8 nodes a wave) x-
// and y-lines then meet no bank twice, z-lines do; without it all three
// directions do (Q7 FP64 with / without: smoothing step 32^3 623 / 644 us, 64^3
// 5.59 / 5.65 ms, apply 64^3 727 / 735 us; FP32 within 1.5%).  No choice of strides
// brings the other degrees as much.
constexpr int SZ = (D == 3) ? E * SY + (n == 8 ? 8 : 0) : 0;
constexpr int TS = (D == 2) ? E * SY : E * SZ;      // padded tile size
constexpr int NF = (D == 2) ? E : E * E;            // nodes of one patch face

// Basis data of Q_K fixed at compile time (instruction immediates); only the
// penalty and the patch eigenpairs come from the Tab struct.
static constexpr ref1d::Ref<K> kRef = ref1d::make_ref<K>();

// threads per patch (one per line) and patches per workgroup
constexpr int TPP = NL;
static_assert(TPP == NL, "each thread owns exactly one line per phase");
constexpr int PPB_DEFAULT = (D == 3)
    ? (K == 1 ? 4 : 1)
    : (K == 1 ? 16 : K == 2 ? 10 : K == 3 ? 8 : K == 4 ? 6 : K == 5 ? 5 : 4);

// base offset and stride of LDS line l along direction dir
__device__ __forceinline__ void line_geom(int dir, int l, int& base, int& stride) {
  const int a = l % E, b = l / E;
  if (dir == 0) { base = a * SY + b * SZ; stride = 1; }
  else if (dir == 1) { base = a + b * SZ; stride = SY; }
  else { base = a + b * SY; stride = SZ; }
}

template <typename T>
struct Line { T v[E]; };

template <typename T>
__device__ __forceinline__ void load_line(const T* s, int base, int stride, Line<T>& L) {
#pragma unroll
  for (int p = 0; p < E; ++p) L.v[p] = s[base + p * stride];
}
template <typename T>
__device__ __forceinline__ void store_line(T* s, int base, int stride, const Line<T>& L) {
#pragma unroll
  for (int p = 0; p < E; ++p) s[base + p * stride] = L.v[p];
}

// Even-odd form of the cell blocks (from Q4 on).  M and the consistency
// block Lcons are symmetric under the reflection of a cell (mu -> n-1-mu,
// nu -> n-1-nu), so B w for a cell line w is formed from sums ve and
// differences vo of mirrored values: the even part e = A ve (+ the middle
// column times the middle value for odd n), the odd part d = Bo vo, outputs
// e + d and e - d at mirrored rows (and the middle row from ve for odd n),
// with A, Bo the half-sums and half-differences of mirrored columns.  Fewer
// multiply-adds: 48 instead of 64 for n = 8.
constexpr bool kEOC = (K >= 4);
constexpr int kHN = n / 2;
constexpr bool kOddN = (n % 2) == 1;
struct EOCell {
  double A[kHN * kHN];
  double Bo[kHN * kHN];
  double colm[kHN + 1];  // middle column (rows < kHN), odd n
  double rowm[kHN + 1];  // middle row (columns < kHN, then the diagonal), odd n
};
constexpr EOCell make_eo_cell(const double (&B)[n * n]) {
  EOCell r{};
  for (int mu = 0; mu < kHN; ++mu)
    for (int j = 0; j < kHN; ++j) {
      r.A[mu * kHN + j] = 0.5 * (B[mu * n + j] + B[mu * n + n - 1 - j]);
      r.Bo[mu * kHN + j] = 0.5 * (B[mu * n + j] - B[mu * n + n - 1 - j]);
    }
  if (kOddN) {
    for (int mu = 0; mu < kHN; ++mu) r.colm[mu] = B[mu * n + kHN];
    for (int j = 0; j < kHN; ++j) r.rowm[j] = B[kHN * n + j];
    r.rowm[kHN] = B[kHN * n + kHN];
  }
  return r;
}
static constexpr EOCell kEOM = make_eo_cell(kRef.M);
static constexpr EOCell kEOL = make_eo_cell(kRef.Lcons);
static constexpr EOCell kEOK = make_eo_cell(kRef.Ks);

// bl = B w for the cell c of patch line v (MASS: B = M, else Lcons)
template <typename T, bool MASS>
__device__ __forceinline__ void cell_eo(const Line<T>& v, int c, T (&bl)[n]) {
  constexpr const EOCell& C = MASS ? kEOM : kEOL;
  T ve[kHN], vo[kHN];
#pragma unroll
  for (int j = 0; j < kHN; ++j) {
    ve[j] = v.v[c * n + j] + v.v[c * n + n - 1 - j];
    vo[j] = v.v[c * n + j] - v.v[c * n + n - 1 - j];
  }
#pragma unroll
  for (int mu = 0; mu < kHN; ++mu) {
    T se = T(0), so = T(0);
#pragma unroll
    for (int j = 0; j < kHN; ++j) se += T(C.A[mu * kHN + j]) * ve[j];
    if constexpr (kOddN) se += T(C.colm[mu]) * v.v[c * n + kHN];
#pragma unroll
    for (int j = 0; j < kHN; ++j) so += T(C.Bo[mu * kHN + j]) * vo[j];
    bl[mu] = se + so;
    bl[n - 1 - mu] = se - so;
  }
  if constexpr (kOddN) {
    T sm = T(0);
#pragma unroll
    for (int j = 0; j < kHN; ++j) sm += T(C.rowm[j]) * ve[j];
    sm += T(C.rowm[kHN]) * v.v[c * n + kHN];
    bl[kHN] = sm;
  }
}

// o = blockdiag(M, M) v; the end outputs o[0] and o[E-1] only when need0 /
// needE (wave-uniform): smoothers drop them on interior patch faces
template <typename T>
__device__ __forceinline__ void line_mass(const Tab<K, T>* __restrict__ t, const Line<T>& v, Line<T>& o,
                                          bool need0 = true, bool needE = true) {
  if constexpr (kEOC) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T bl[n];
      cell_eo<T, true>(v, c, bl);
#pragma unroll
      for (int mu = 0; mu < n; ++mu) {
        const int p = c * n + mu;
        if ((p == 0 && !need0) || (p == E - 1 && !needE)) continue;
        o.v[p] = bl[mu];
      }
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int mu = 0; mu < n; ++mu) {
      const int p = c * n + mu;
      if ((p == 0 && !need0) || (p == E - 1 && !needE)) continue;
      T s = T(0);
#pragma unroll
      for (int nu = 0; nu < n; ++nu) s += T(kRef.M[mu * n + nu]) * v.v[c * n + nu];
      o.v[p] = s;
    }
}

// 1/x from the hardware reciprocal estimate refined by one Newton step
// r <- r (2 - x r); the squared relative error of the estimate is far below
// the FP64 tolerance of the smoother.  x is a positive finite sum of patch
// eigenvalues (unused slots carry a huge finite value, giving ~0).
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return __builtin_fmaf(r, __builtin_fmaf(-x, r, 1.0f), r);
}

// Couplings of a patch line to what lies beyond its two outer faces.
template <typename T>
struct Sides {
  bool bl, br;   // left / right outer face on the domain boundary (Nitsche)
  T aL, bL, aR, bR;  // interior-neighbour couplings (ignored on boundary sides)
  // the paper's Dirichlet residual: on interior outer faces leave out the
  // consistency term -[[u]].{grad v} altogether (its inside half, carried by
  // the cell block, is cancelled from the line's own end value)
  bool lit;
};

// FP32 evaluates the 1-D operator on differences: stiffness and end derivatives
// of a cell act on its values less one of them (their rows sum to zero, so a
// column drops out), the face terms on jumps.  With the values themselves the
// rounding of the coefficients acts like a small reaction term: the FP32
// V-cycles of Q5..Q7 on random loads were off by 1e-6..4e-5.  The shortest lines
// keep the plain rows: 2-D Q1, and 3-D up to Q3, whose V-cycles on plain rows
// are off by 2e-7..7e-7 (on differences 2e-7..5e-7) and whose FP32 operator is
// 3-6% faster on them (3-D Q3 8^3 4.13 / 4.39 us, 32^3 8.1 / 8.4 us, Q1 64^3
// restriction 11.1 / 11.8 us); 2-D Q2, Q3 would be off by up to 1.6e-6.  FP64
// keeps the plain rows.  One apply on random values is off by 2-7% more on
// differences, for their own rounding (3-D Q5 9.7e-8 / 9.3e-8).
template <typename T>
constexpr bool kDiff = sizeof(T) == 4 && K >= (D == 3 ? 4 : 2);

// alpha of a face from the neighbour's derivative g and trace tr; on
// differences the penalty part is left to the line, which forms the jump
template <typename T, int SIDE>
__device__ __forceinline__ T face_alpha(T sg, T g, T tr) {
  const T half = T(0.5);
  if constexpr (kDiff<T>) return SIDE == 0 ? half * g : -half * g;
  else return SIDE == 0 ? (half * g - sg * tr) : (-sg * tr - half * g);
}
// end derivative (SIDE 0: d1, the neighbour below; 1: d0, above) of the n
// values w(j) of a neighbour's line
template <typename T, int SIDE, typename W>
__device__ __forceinline__ T face_grad(W w) {
  T g = T(0);
  if constexpr (kDiff<T>) {
    const T w0 = w(0);
#pragma unroll
    for (int j = 1; j < n; ++j) g += (SIDE == 0 ? T(kRef.d1[j]) : T(kRef.d0[j])) * (w(j) - w0);
  } else {
#pragma unroll
    for (int j = 0; j < n; ++j) g += (SIDE == 0 ? T(kRef.d1[j]) : T(kRef.d0[j])) * w(j);
  }
  return g;
}
// end derivatives of cell c of a line (at its left and right end), on
// differences: the even and odd parts serve both
template <typename T>
__device__ __forceinline__ void cell_grad(const Line<T>& v, int c, T& g0, T& g1) {
  const T ref = kOddN ? v.v[c * n + kHN] + v.v[c * n + kHN] : v.v[c * n] + v.v[c * n + n - 1];
  T e = T(0), o = T(0);
#pragma unroll
  for (int j = kOddN ? 0 : 1; j < kHN; ++j)
    e += T(0.5 * (kRef.d0[j] + kRef.d0[n - 1 - j])) * ((v.v[c * n + j] + v.v[c * n + n - 1 - j]) - ref);
#pragma unroll
  for (int j = 0; j < kHN; ++j)
    o += T(0.5 * (kRef.d0[j] - kRef.d0[n - 1 - j])) * (v.v[c * n + j] - v.v[c * n + n - 1 - j]);
  g0 = o + e;
  g1 = o - e;
}
// stiffness rows of cell c of a line, on differences
template <typename T>
__device__ __forceinline__ void cell_stiff(const Line<T>& v, int c, T (&bl)[n]) {
  const T ref = kOddN ? v.v[c * n + kHN] + v.v[c * n + kHN] : v.v[c * n] + v.v[c * n + n - 1];
  T ve[kHN], vo[kHN];
#pragma unroll
  for (int j = 0; j < kHN; ++j) {
    ve[j] = (v.v[c * n + j] + v.v[c * n + n - 1 - j]) - ref;
    vo[j] = v.v[c * n + j] - v.v[c * n + n - 1 - j];
  }
#pragma unroll
  for (int mu = 0; mu < kHN; ++mu) {
    T se = T(0), so = T(0);
#pragma unroll
    for (int j = kOddN ? 0 : 1; j < kHN; ++j) se += T(kEOK.A[mu * kHN + j]) * ve[j];
#pragma unroll
    for (int j = 0; j < kHN; ++j) so += T(kEOK.Bo[mu * kHN + j]) * vo[j];
    bl[mu] = se + so;
    bl[n - 1 - mu] = se - so;
  }
  if constexpr (kOddN) {
    T sm = T(0);
#pragma unroll
    for (int j = 0; j < kHN; ++j) sm += T(kEOK.rowm[j]) * ve[j];
    bl[kHN] = sm;
  }
}
// The face at the outer left (SIDE 0) or right end of a patch line, on
// differences: what it adds to the end row (end) and the factor of d0 (d1) it
// adds to the rows of its cell (cf); v0: the line's end value, g: the line's
// derivative there.
template <typename T, int SIDE>
__device__ __forceinline__ void outer_face(T sg, const Sides<T>& sd, T v0, T g, T& end, T& cf) {
  const T half = T(0.5);
  const bool bnd = SIDE == 0 ? sd.bl : sd.br;
  const T gs = SIDE == 0 ? g : -g;
  if (bnd) {  // Nitsche: no value beyond
    end = sg * v0 + gs;
    cf = SIDE == 0 ? v0 : -v0;
  } else if (sd.lit) {
    end = sg * v0 + half * gs;
    cf = T(0);
  } else {
    const T jump = SIDE == 0 ? v0 + (sd.bL + sd.bL) : v0 - (sd.bR + sd.bR);  // own less the neighbour's
    end = sg * jump + ((SIDE == 0 ? sd.aL : sd.aR) + half * gs);
    cf = SIDE == 0 ? half * jump : -half * jump;
  }
}
// rows of cell C of the patch line v, on differences
template <typename T, int C, bool ACC>
__device__ __forceinline__ void cell_sipg_diff(T sg, const Line<T>& v, const Sides<T>& sd, T (&o)[n], bool need0,
                                               bool needE) {
  const T half = T(0.5);
  T g00, g01, g10, g11, bl[n];
  cell_grad<T>(v, 0, g00, g01);
  cell_grad<T>(v, 1, g10, g11);
  cell_stiff<T>(v, C, bl);
  // the face between the two cells
  const T jump = v.v[n - 1] - v.v[n];
  const T mid = sg * jump - half * (g01 + g10);
  T end, cf;
  if constexpr (C == 0) outer_face<T, 0>(sg, sd, v.v[0], g00, end, cf);
  else outer_face<T, 1>(sg, sd, v.v[E - 1], g11, end, cf);
  const T c0 = C == 0 ? cf : -half * jump;  // factor of d0 (left face of the cell)
  const T c1 = C == 0 ? -half * jump : cf;  // factor of d1
#pragma unroll
  for (int mu = 0; mu < n; ++mu) {
    if ((C == 0 && mu == 0 && !need0) || (C == 1 && mu == n - 1 && !needE)) continue;
    T s = ACC ? o[mu] : T(0);
    s += bl[mu];
    if (mu == 0) s += C == 0 ? end : -mid;
    if (mu == n - 1) s += C == 0 ? mid : end;
    s += T(kRef.d0[mu]) * c0 + T(kRef.d1[mu]) * c1;
    o[mu] = s;
  }
}

// o (+)= 1-D SIPG of the patch line v; the end outputs only when need0 / needE
template <typename T, bool ACC>
__device__ __forceinline__ void line_sipg(const Tab<K, T>* __restrict__ t, const Line<T>& v,
                                          const Sides<T>& sd, Line<T>& o, bool need0 = true,
                                          bool needE = true) {
  if constexpr (kDiff<T>) {
    T lo[n], hi[n];
    if constexpr (ACC) {
#pragma unroll
      for (int mu = 0; mu < n; ++mu) {
        lo[mu] = o.v[mu];
        hi[mu] = o.v[n + mu];
      }
    }
    cell_sipg_diff<T, 0, ACC>(t->sigma, v, sd, lo, need0, needE);
    cell_sipg_diff<T, 1, ACC>(t->sigma, v, sd, hi, need0, needE);
#pragma unroll
    for (int mu = 0; mu < n; ++mu) {
      if (mu > 0 || need0) o.v[mu] = lo[mu];
      if (mu < n - 1 || needE) o.v[n + mu] = hi[mu];
    }
    return;
  }
  const T sg = t->sigma;
  const T half = T(0.5);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    T bl[n];
    if constexpr (kEOC) cell_eo<T, false>(v, c, bl);
#pragma unroll
    for (int mu = 0; mu < n; ++mu) {
      const int p = c * n + mu;
      if ((p == 0 && !need0) || (p == E - 1 && !needE)) continue;
      T s = ACC ? o.v[p] : T(0);
      if constexpr (kEOC) {
        s += bl[mu];
      } else {
#pragma unroll
        for (int nu = 0; nu < n; ++nu) s += T(kRef.Lcons[mu * n + nu]) * v.v[c * n + nu];
      }
      if (mu == 0) s += sg * v.v[c * n];          // penalty part of the cell block
      if (mu == n - 1) s += sg * v.v[c * n + n - 1];
      o.v[p] = s;
    }
  }
  // face between the two patch cells
  const T tR = v.v[n];      // trace of the right cell at its x=0 side
  const T tL = v.v[n - 1];  // trace of the left cell at its x=1 side
  T gR = T(0), gL = T(0);
#pragma unroll
  for (int j = 0; j < n; ++j) {
    gR += T(kRef.d0[j]) * v.v[n + j];
    gL += T(kRef.d1[j]) * v.v[j];
  }
  T aL = sd.aL, bL = sd.bL, aR = sd.aR, bR = sd.bR;
  if (sd.bl) {  // Nitsche correction of the left cell (uniform per patch)
    T g0 = T(0);
#pragma unroll
    for (int j = 0; j < n; ++j) g0 += T(kRef.d0[j]) * v.v[j];
    aL = half * g0;
    bL = half * v.v[0];
  }
  if (sd.br) {
    T g1 = T(0);
#pragma unroll
    for (int j = 0; j < n; ++j) g1 += T(kRef.d1[j]) * v.v[n + j];
    aR = -half * g1;
    bR = -half * v.v[E - 1];
  }
  if (!sd.bl && sd.lit) bL = -half * v.v[0];
  if (!sd.br && sd.lit) bR = half * v.v[E - 1];
  const T bLc = half * tR;   // beta seen by the left cell from its right neighbour
  const T bRc = -half * tL;  // beta seen by the right cell from its left neighbour
  if (need0) {
    o.v[0] += aL;
    o.v[0] += T(kRef.d0[0]) * bL + T(kRef.d1[0]) * bLc;
  }
  o.v[n - 1] += -sg * tR - half * gR;
  o.v[n] += half * gL - sg * tL;
  if (needE) {
    o.v[E - 1] += aR;
    o.v[E - 1] += T(kRef.d0[n - 1]) * bRc + T(kRef.d1[n - 1]) * bR;
  }
#pragma unroll
  for (int mu = 0; mu < n; ++mu) {
    if (mu > 0) o.v[mu] += T(kRef.d0[mu]) * bL + T(kRef.d1[mu]) * bLc;
    if (mu < n - 1) o.v[n + mu] += T(kRef.d0[mu]) * bRc + T(kRef.d1[mu]) * bR;
  }
}

// Fast-diagonalisation contractions for patch type TY of a local space SP:
// SP_DIR the Dirichlet space, SP_FULL the whole patch, SP_CLAMPED the clamped
// space (tables C S).  Padded S: rows p in [PLO, PHI) and columns q < QN are
// the only non-zeros.
constexpr int SP_DIR = 0, SP_FULL = 1, SP_CLAMPED = 2;
template <int SP, int TY> struct FDB;
template <> struct FDB<SP_DIR, 0> { static constexpr int PLO = 1, PHI = E - 1, QN = E - 2; };
template <> struct FDB<SP_DIR, 1> { static constexpr int PLO = 0, PHI = E - 1, QN = E - 1; };
template <> struct FDB<SP_DIR, 2> { static constexpr int PLO = 1, PHI = E, QN = E - 1; };
template <> struct FDB<SP_DIR, 3> { static constexpr int PLO = 0, PHI = E, QN = E; };
template <int TY> struct FDB<SP_FULL, TY> { static constexpr int PLO = 0, PHI = E, QN = E; };
// clamped: value and derivative fixed at each interior-face end (two
// unknowns fewer per clamped end; the end node itself stays zero)
template <> struct FDB<SP_CLAMPED, 0> { static constexpr int PLO = 1, PHI = E - 1, QN = E - 4; };
template <> struct FDB<SP_CLAMPED, 1> { static constexpr int PLO = 0, PHI = E - 1, QN = E - 2; };
template <> struct FDB<SP_CLAMPED, 2> { static constexpr int PLO = 1, PHI = E, QN = E - 2; };
template <> struct FDB<SP_CLAMPED, 3> { static constexpr int PLO = 0, PHI = E, QN = E; };

// The 1-D data of one pass.  OPQ: through a pointer the compiler cannot connect
// with other passes' reads of the same table.  Otherwise it keeps the
// coefficients of one pass (up to E^2) for the next in scalar registers it
// does not have, and every pass spends more instructions on spilling them to
// vector lanes than on arithmetic.  Constant address space: scalar loads.
template <typename T>
using Coef = const T __attribute__((address_space(4)))*;
template <typename T, bool OPQ>
__device__ __forceinline__ Coef<T> pass_coef(const T* p) {
  unsigned long long a = (unsigned long long)p;
  if constexpr (OPQ) asm volatile("" : "+s"(a));
  return (Coef<T>)a;
}

template <typename T, int SP>
__device__ __forceinline__ const T* fd_S(const Tab<K, T>* __restrict__ t, int ty) {
  return SP == SP_FULL ? t->Sf[ty] : SP == SP_CLAMPED ? t->Sc[ty] : t->S[ty];
}
template <typename T, int SP>
__device__ __forceinline__ const T* fd_lam(const Tab<K, T>* __restrict__ t, int ty) {
  return SP == SP_FULL ? t->lamf[ty] : SP == SP_CLAMPED ? t->lamc[ty] : t->lam[ty];
}
// Inverse eigenvalue sums of the scaling line of a lane (3-D: the y-line
// (qx, qz) = (l % E, l / E); 2-D: the x-line qy = l): E values from the
// patch-type combination's table, read at the start of a colour step so that
// the loads overlap the operator passes.
template <typename T, int SP>
__device__ __forceinline__ void load_rs(const Tab<K, T>* __restrict__ t, const int (&ty)[3], int l,
                                        T (&r)[E]) {
  const int combo = (D == 3) ? (ty[0] * 4 + ty[1]) * 4 + ty[2] : ty[0] * 4 + ty[1];
  const T* p = t->rs[SP == SP_FULL ? 1 : SP == SP_CLAMPED ? 2 : 0][combo + (D == 2 && SP == SP_DIR ? 16 : 0)] + l * E;
#pragma unroll
  for (int q = 0; q < E; ++q) r[q] = p[q];
}

// Interior patches (type 0) on the Dirichlet space: the 1-D problem is
// symmetric under the reflection p -> E-1-p, and the host computes its
// eigenvectors on the even and the odd subspace (columns q < h even,
// h <= q < 2h odd, h = n - 1).  S^T then contracts sums v+ and differences v-
// of mirrored nodes with half columns, and S forms the even part e and odd
// part d of each mirrored pair: 2 h^2 multiply-adds instead of 4 h^2 (a wave of
// an interior Q3 patch in FP64: 970 vector instructions without, 472 with it
// and the compile-time patch type).
constexpr int kEOH = n - 1;
constexpr bool kEO = (K >= 2);

template <typename T>
__device__ __forceinline__ void eo_split(const Line<T>& v, T (&vp)[kEOH], T (&vm)[kEOH]) {
#pragma unroll
  for (int k = 0; k < kEOH; ++k) {
    vp[k] = v.v[1 + k] + v.v[E - 2 - k];
    vm[k] = v.v[1 + k] - v.v[E - 2 - k];
  }
}
// coefficient q < 2h of S^T v
template <typename T>
__device__ __forceinline__ T eo_coef(Coef<T> S, const T (&vp)[kEOH], const T (&vm)[kEOH], int q) {
  T s = T(0);
#pragma unroll
  for (int k = 0; k < kEOH; ++k) s += S[(1 + k) * E + q] * (q < kEOH ? vp[k] : vm[k]);
  return s;
}
// even and odd parts of the outputs at nodes 1 + k and E - 2 - k of S v
template <typename T>
__device__ __forceinline__ void eo_pair(Coef<T> S, const Line<T>& v, int k, T& e, T& d) {
  T se = T(0), sd = T(0);
#pragma unroll
  for (int q = 0; q < kEOH; ++q) se += S[(1 + k) * E + q] * v.v[q];
#pragma unroll
  for (int q = 0; q < kEOH; ++q) sd += S[(1 + k) * E + kEOH + q] * v.v[kEOH + q];
  e = se;
  d = sd;
}

// Which spaces' contractions read S opaquely (pass_coef): all of the Dirichlet
// space; of the larger ones those whose table does not fit the scalar
// registers and whose patch type the compiler knows to be uniform in a wave --
// elsewhere it reads the types' tables ahead of the diverging branches, and
// that is worth more (smoothing steps of the Full kernel on 32^3, opaque
// against not: Q7 FP32 726 / 1322 us, Q3 FP64 156 / 185 us, but Q2 FP64 189 /
// 173 us, Q4 FP64 1002 / 924 us).
template <typename T, int SP>
constexpr bool kOpaqueFD = SP == SP_DIR || (TPP % 64 == 0 && E * E * (int)sizeof(T) > 4 * 100);

// o[q] = sum_p S[p][q] v[p]
template <typename T, int TY, int SP>
__device__ __forceinline__ void line_St_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, Line<T>& o) {
  using B = FDB<SP, TY>;
  const Coef<T> S = pass_coef<T, kOpaqueFD<T, SP>>(fd_S<T, SP>(t, TY));
  if constexpr (kEO && SP == SP_DIR && TY == 0) {
    T vp[kEOH], vm[kEOH];
    eo_split<T>(v, vp, vm);
#pragma unroll
    for (int q = 0; q < E; ++q) o.v[q] = (q < 2 * kEOH) ? eo_coef<T>(S, vp, vm, q) : T(0);
    return;
  }
#pragma unroll
  for (int q = 0; q < E; ++q) {
    T s = T(0);
    if (q < B::QN) {
#pragma unroll
      for (int p = B::PLO; p < B::PHI; ++p) s += S[p * E + q] * v.v[p];
    }
    o.v[q] = s;
  }
}
// o[p] = sum_q S[p][q] v[q]
template <typename T, int TY, int SP>
__device__ __forceinline__ void line_S_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, Line<T>& o) {
  using B = FDB<SP, TY>;
  const Coef<T> S = pass_coef<T, kOpaqueFD<T, SP>>(fd_S<T, SP>(t, TY));
  if constexpr (kEO && SP == SP_DIR && TY == 0) {
    // outputs written in increasing node order, as in the other types: the
    // compiler then merges the four type branches' stores into one line
    // without a runtime-indexed copy of it (which would live in scratch)
    T e[kEOH], d[kEOH];
#pragma unroll
    for (int k = 0; k < kEOH; ++k) eo_pair<T>(S, v, k, e[k], d[k]);
    o.v[0] = T(0);
#pragma unroll
    for (int k = 0; k < kEOH; ++k) o.v[1 + k] = e[k] + d[k];
#pragma unroll
    for (int k = kEOH - 1; k >= 0; --k) o.v[E - 2 - k] = e[k] - d[k];
    o.v[E - 1] = T(0);
    return;
  }
#pragma unroll
  for (int p = 0; p < E; ++p) {
    T s = T(0);
    if (p >= B::PLO && p < B::PHI) {
#pragma unroll
      for (int q = 0; q < B::QN; ++q) s += S[p * E + q] * v.v[q];
    }
    o.v[p] = s;
  }
}
template <typename T, int SP>
__device__ __forceinline__ void line_St(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v, Line<T>& o) {
  switch (ty) {
    case 0: line_St_t<T, 0, SP>(t, v, o); break;
    case 1: line_St_t<T, 1, SP>(t, v, o); break;
    case 2: line_St_t<T, 2, SP>(t, v, o); break;
    default: line_St_t<T, 3, SP>(t, v, o); break;
  }
}
template <typename T, int SP>
__device__ __forceinline__ void line_S(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v, Line<T>& o) {
  switch (ty) {
    case 0: line_S_t<T, 0, SP>(t, v, o); break;
    case 1: line_S_t<T, 1, SP>(t, v, o); break;
    case 2: line_S_t<T, 2, SP>(t, v, o); break;
    default: line_S_t<T, 3, SP>(t, v, o); break;
  }
}

// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).
// Renumber them so that XCD j works on the j-th contiguous range of patches:
// neighbouring patches, whose face traces a patch reads, then sit in the
// same L2.  Bijective on [0, nblocks).
__device__ __forceinline__ int xcd_block(int b, int nblocks, int remap) {
  if (!remap || nblocks < 8) return b;
  const int q = nblocks / 8, r = nblocks % 8;
  const int xcd = b % 8, idx = b / 8;
  return xcd * q + (xcd < r ? xcd : r) + idx;
}

// Workgroup slot of the calling thread (TPP threads per slot): a scalar
// where a slot spans whole waves, so that the patch index and position that
// follow from it stay in scalar registers.
__device__ __forceinline__ int slot_of() {
  const int s = (int)threadIdx.x / TPP;
  if constexpr (TPP % 64 == 0) return __builtin_amdgcn_readfirstlane(s);
  return s;
}

// Patch and right-hand side of workgroup slot `slot`: PPB patches of one
// right-hand side per workgroup, or (RP, right-hand-side packing) one patch
// for PPB consecutive right-hand sides, so that every slot of the workgroup
// has the same patch type and position (uniform branches and scalar loads of
// the 1-D data where slots share a wave); slots past the last right-hand side
// get an out-of-range patch index, npatch more than the others', and only meet
// the barriers.
template <int PPB, bool RP>
__device__ __forceinline__ void slot_work(const PatchGrid& g, int slot, int& pid, int& rhs) {
  const int blk = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap);
  if constexpr (RP) {
    rhs = (int)blockIdx.y * PPB + slot;
    pid = rhs < g.nrhs ? blk : blk + g.npatch;
    if (rhs >= g.nrhs) rhs = 0;
  } else {
    pid = blk * PPB + slot;
    rhs = blockIdx.y;
  }
}

// Patch coordinates of patch index pid of a launch.
struct PatchPos {
  int lo[3];
  int ty[3];  // 1-D patch type: bit 0 touches x_i = 0, bit 1 touches x_i = 1
};
__device__ __forceinline__ PatchPos patch_pos(const PatchGrid& g, int pid) {
  PatchPos P;
  int r = pid;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (i < D) {
      // r / cnt by the launch's multiplier (grid_magic); the last quotient is 0
      int quo = 0;
      if (i < D - 1) quo = g.mul[i] ? (int)__umulhi((unsigned)r, g.mul[i]) : r / g.cnt[i];
      const int m = r - quo * g.cnt[i];
      r = quo;
      P.lo[i] = g.off[i] + 2 * m;
      const int v = P.lo[i] + 1;  // the patch's vertex
      P.ty[i] = (v == 1 ? 1 : 0) | (v == g.N - 1 ? 2 : 0);
    } else {
      P.lo[i] = 0;
      P.ty[i] = 0;
    }
  }
  return P;
}

__device__ __forceinline__ long long cell_index(int N, int cx, int cy, int cz) {
  return (long long)cx + (long long)N * ((long long)cy + (long long)N * (long long)cz);
}

// Global offset of tile node (px, py, pz) of the patch.
__device__ __forceinline__ long long node_offset(int N, const PatchPos& P, int px, int py, int pz) {
  const int cx = px / n, ax = px % n;
  const int cy = py / n, ay = py % n;
  const int cz = (D == 3) ? pz / n : 0, az = (D == 3) ? pz % n : 0;
  const long long cell = cell_index(N, P.lo[0] + cx, P.lo[1] + cy, (D == 3) ? P.lo[2] + cz : 0);
  return cell * NC + ax + n * (ay + n * az);
}

// Global offset of the first node of the patch's x-line (py, pz) (cell lo_x).
__device__ __forceinline__ long long xrow_offset(int N, const PatchPos& P, int py, int pz) {
  return node_offset(N, P, 0, py, (D == 3) ? pz : 0);
}

// Side flags and x-face couplings of an x-line for the full operator from the
// n values of the rows of its outside x-neighbours (rl: the cell below, rr:
// the cell above; ignored on boundary sides).
template <typename T>
__device__ __forceinline__ Sides<T> xsides_rows(T sg, bool bl, bool br, const T (&rl)[n], const T (&rr)[n]) {
  const T half = T(0.5);
  Sides<T> sd;
  sd.bl = bl;
  sd.br = br;
  sd.aL = sd.bL = sd.aR = sd.bR = T(0);
  sd.lit = false;
  if (!sd.bl) {
    const T tr = rl[K];
    sd.bL = -half * tr;
    sd.aL = face_alpha<T, 0>(sg, face_grad<T, 0>([&](int j) { return rl[j]; }), tr);
  }
  if (!sd.br) {
    const T tr = rr[0];
    sd.bR = half * tr;
    sd.aR = face_alpha<T, 1>(sg, face_grad<T, 1>([&](int j) { return rr[j]; }), tr);
  }
  return sd;
}

// Side flags of a line with cells lo, lo + 1 of N along it and no data beyond
template <typename T>
__device__ __forceinline__ Sides<T> bare_sides(int lo, int N, bool lit) {
  return Sides<T>{lo == 0, lo + 1 == N - 1, T(0), T(0), T(0), T(0), lit};
}

// Side flags and x-face couplings of an operator x-line (py, pz), read from the
// rows of the outside neighbours.
template <typename T>
__device__ __forceinline__ Sides<T> xline_sides(const Tab<K, T>* __restrict__ t, const T* __restrict__ x,
                                                int N, const PatchPos& P, long long row0) {
  const T half = T(0.5);
  const T sg = t->sigma;
  Sides<T> sd = bare_sides<T>(P.lo[0], N, false);
  if (!sd.bl) {
    const T* r = x + row0 - NC;
    const T tr = r[K];
    sd.bL = -half * tr;
    sd.aL = face_alpha<T, 0>(sg, face_grad<T, 0>([&](int j) { return r[j]; }), tr);
  }
  if (!sd.br) {
    const T* r = x + row0 + 2 * NC;
    const T tr = r[0];
    sd.bR = half * tr;
    sd.aR = face_alpha<T, 1>(sg, face_grad<T, 1>([&](int j) { return r[j]; }), tr);
  }
  return sd;
}

// Raw face data (alpha, beta) of interior neighbours across y- (and z-) faces for
// the operator.  Entry i enumerates (dir, side, face node f); f = a + E b with
// (a, b) the tangential patch coordinates in increasing direction order.  Layout:
// ext[(fd * 2 + side) * 2 + comp][f] with fd = dir - 1.
template <typename T>
__device__ __forceinline__ void gather_ext(const Tab<K, T>* __restrict__ t, const T* __restrict__ x,
                                           int N, const PatchPos& P, int lane, T* ext) {
  const T half = T(0.5);
  const T sg = t->sigma;
  // a patch face has one node per lane (NF = TPP), so entry block it = fd * 2 +
  // side holds this lane's face node f = lane: unrolled, direction and side are
  // compile-time constants of each block
  static_assert(NF == TPP, "one face node per lane");
#pragma unroll
  for (int it = 0; it < (D - 1) * 2; ++it) {
    const int f = lane;
    const int side = it & 1;
    const int fd = it / 2;
    const int dir = fd + 1;
    const int lod = (dir == 1) ? P.lo[1] : P.lo[2];  // not P.lo[dir]: no scratch copy of P
    const int nb = (side == 0) ? lod - 1 : lod + 2;
    T alpha = T(0), beta = T(0);
    if (nb >= 0 && nb < N) {
      // neighbour cell and the face node's local coordinates in it (tangential
      // coordinates from (a, b), 0 along dir); named per direction rather than
      // indexed by the runtime dir, which would put the arrays in scratch
      const int a = f % E, b = f / E;
      const int cx = P.lo[0] + a / n, ax = a % n;
      const int cy = (dir == 1) ? nb : P.lo[1] + b / n, ay = (dir == 1) ? 0 : b % n;
      const int cz = (D == 2) ? 0 : (dir == 1) ? P.lo[2] + b / n : nb;
      const int az = (D == 2 || dir != 1) ? 0 : b % n;
      const int strideN = (dir == 1) ? n : n * n;
      const long long base = cell_index(N, cx, cy, cz) * NC + ax + n * (ay + n * az);
      const T tr = x[base + (long long)((side == 0) ? K : 0) * strideN];
      beta = (side == 0) ? -half * tr : half * tr;
      auto w = [&](int j) { return x[base + (long long)j * strideN]; };
      alpha = (side == 0) ? face_alpha<T, 0>(sg, face_grad<T, 0>(w), tr)
                          : face_alpha<T, 1>(sg, face_grad<T, 1>(w), tr);
    }
    ext[((fd * 2 + side) * 2 + 0) * NF + f] = alpha;
    ext[((fd * 2 + side) * 2 + 1) * NF + f] = beta;
  }
}

// row[nu] = M[mu][nu] for a lane-dependent mu, read from a device copy of
// the mass matrix (n vector loads instead of a select chain per entry)
template <typename T>
struct MassRows {
  T v[n * n];
};
template <typename T>
constexpr MassRows<T> make_mass_rows() {
  MassRows<T> r{};
  for (int i = 0; i < n * n; ++i) r.v[i] = T(kRef.M[i]);
  return r;
}
template <typename T>
__device__ constexpr MassRows<T> kMassRows = make_mass_rows<T>();

template <typename T>
__device__ __forceinline__ void mass_row(int mu, T (&row)[n]) {
#pragma unroll
  for (int nu = 0; nu < n; ++nu) row[nu] = kMassRows<T>.v[mu * n + nu];
}

// The mass row that contracts the neighbours' face data.  On differences (FP32)
// it acts as the line's own mass does (line_mass), in the same operations:
// rounded another way, the two sides' masses would leave a jump that the
// penalty multiplies.  With the even-odd form (kFaceEO) a row holds its half-sums
// (n / 2), its half-differences (negative in the mirrored rows) and, for odd n, the
// coefficient of the middle value, each rounded once: rows and even-odd form on one
// coarser grid of coefficients instead put the 3-D FP32 operator off by 1.41e-7
// (Q5), 1.15e-7 (Q6), 1.25e-7 (Q7) on uniform random values, in this form 9.7e-8, 9.5e-8,
// 9.9e-8.  Elsewhere the plain rows, as mass_row.
template <typename T>
constexpr bool kFaceEO = kDiff<T> && kEOC;
template <typename T>
constexpr MassRows<T> make_face_rows() {
  MassRows<T> r = make_mass_rows<T>();
  if (kFaceEO<T>)
    for (int mu = 0; mu < n; ++mu) {
      const int m = mu < n - 1 - mu ? mu : n - 1 - mu;
      const bool mid = kOddN && mu == kHN;
      for (int j = 0; j < kHN; ++j) {
        r.v[mu * n + j] = T(mid ? kEOM.rowm[j] : kEOM.A[m * kHN + j]);
        r.v[mu * n + kHN + j] = T(mid ? 0.0 : mu == m ? kEOM.Bo[m * kHN + j] : -kEOM.Bo[m * kHN + j]);
      }
      if (kOddN) r.v[mu * n + n - 1] = T(mid ? kEOM.rowm[kHN] : kEOM.colm[m]);
    }
  return r;
}
template <typename T>
__device__ constexpr MassRows<T> kFaceRows = make_face_rows<T>();
template <typename T>
__device__ __forceinline__ void face_row(int mu, T (&row)[n]) {
#pragma unroll
  for (int nu = 0; nu < n; ++nu) row[nu] = kFaceRows<T>.v[mu * n + nu];
}
// sum_nu M[mu][nu] w(nu) for the row of mu
template <typename T, typename W>
__device__ __forceinline__ T face_dot(const T (&row)[n], W w) {
  T s = T(0);
  if constexpr (kFaceEO<T>) {
    T v[n], d = T(0);
#pragma unroll
    for (int nu = 0; nu < n; ++nu) v[nu] = w(nu);
#pragma unroll
    for (int j = 0; j < kHN; ++j) s += row[j] * (v[j] + v[n - 1 - j]);
    if constexpr (kOddN) s += row[n - 1] * v[kHN];
#pragma unroll
    for (int j = 0; j < kHN; ++j) d += row[kHN + j] * (v[j] - v[n - 1 - j]);
    return s + d;
  }
#pragma unroll
  for (int nu = 0; nu < n; ++nu) s += row[nu] * w(nu);
  return s;
}

// mass-contract ext entries along the first tangential coordinate for the
// value at (a, b): sum over the cell block of a
template <typename T>
__device__ __forceinline__ T ext_mx(const Tab<K, T>* __restrict__ t, const T* arr, int a, int b) {
  const int c0 = (a / n) * n, mu = a % n;
  T row[n];
  face_row<T>(mu, row);
  return face_dot<T>(row, [&](int nu) { return arr[c0 + nu + E * b]; });
}
template <typename T>
__device__ __forceinline__ T ext_my(const Tab<K, T>* __restrict__ t, const T* arr, int a, int b) {
  const int c0 = (b / n) * n, mu = b % n;
  T row[n];
  face_row<T>(mu, row);
  return face_dot<T>(row, [&](int nu) { return arr[a + E * (c0 + nu)]; });
}

// Sides of a y-line (px, pz) (D = 3) or (px) (D = 2): ext_y contracted with M_x.
template <typename T>
__device__ __forceinline__ Sides<T> yline_sides(const Tab<K, T>* __restrict__ t, const T* ext,
                                                int N, const PatchPos& P, int px, int pz) {
  Sides<T> sd = bare_sides<T>(P.lo[1], N, false);
  if (!sd.bl) { sd.aL = ext_mx<T>(t, ext + 0 * NF, px, pz); sd.bL = ext_mx<T>(t, ext + 1 * NF, px, pz); }
  if (!sd.br) { sd.aR = ext_mx<T>(t, ext + 2 * NF, px, pz); sd.bR = ext_mx<T>(t, ext + 3 * NF, px, pz); }
  return sd;
}

// Sides of the smoother's y-line (px, pz): the traces of the y-neighbours at
// nodes (a, k or 0, pz), a in the cell block of px, contracted with M_x
// straight from global memory (n contiguous values per side).  MODE 2 (the
// paper's Dirichlet residual) ignores interior neighbours.  Split into the
// loads (yside_load: the mass row and both neighbours' n traces, the patch's
// own cells standing in for a missing neighbour, whose values go unused) and
// the arithmetic (yside_finish), so that callers can issue the loads together
// with their other global loads.
template <typename T>
struct YSideRaw {
  T row[n], l[n], r[n];
};
template <typename T, int MODE>
__device__ __forceinline__ void yside_load(const T* __restrict__ x, int N, const PatchPos& P, int px, int pz,
                                           YSideRaw<T>& y) {
  if (MODE == 2) return;
  const int cx = P.lo[0] + px / n;
  const int cz = (D == 3) ? P.lo[2] + pz / n : 0;
  const int az = (D == 3) ? pz % n : 0;
  const bool bl = (P.lo[1] == 0), br = (P.lo[1] + 1 == N - 1);
  face_row<T>(px % n, y.row);
  const T* rl = x + cell_index(N, cx, bl ? P.lo[1] : P.lo[1] - 1, cz) * NC + K * n + az * n * n;
  const T* rr = x + cell_index(N, cx, br ? P.lo[1] + 1 : P.lo[1] + 2, cz) * NC + az * n * n;
#pragma unroll
  for (int nu = 0; nu < n; ++nu) {
    y.l[nu] = rl[nu];
    y.r[nu] = rr[nu];
  }
}
template <typename T, int MODE>
__device__ __forceinline__ Sides<T> yside_finish(const YSideRaw<T>& y, int N, const PatchPos& P) {
  Sides<T> sd = bare_sides<T>(P.lo[1], N, MODE == 2);
  if (MODE == 2) return sd;
  const T half = T(0.5);
  if (!sd.bl) {
    sd.bL = -half * face_dot<T>(y.row, [&](int nu) { return y.l[nu]; });
  }
  if (!sd.br) {
    sd.bR = half * face_dot<T>(y.row, [&](int nu) { return y.r[nu]; });
  }
  return sd;
}

// In the y-phase the z-face arrays (after the y-face arrays) are contracted along
// x in place (lines at fixed py); in the z-phase the value at (px, py) is
// contracted along y.
template <typename T>
__device__ __forceinline__ void extz_mass_x_line(const Tab<K, T>* __restrict__ t, T* ext, int j) {
  const int py = j % E;
  const int arr = j / E;  // (side * 2 + comp)
  T* a = ext + 4 * NF + arr * NF + py * E;
  T v[E];
#pragma unroll
  for (int p = 0; p < E; ++p) v[p] = a[p];
  // face rows (face data, contracted the same way wherever it is used)
  constexpr MassRows<T> rows = make_face_rows<T>();
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int mu = 0; mu < n; ++mu) {
      T row[n];
#pragma unroll
      for (int nu = 0; nu < n; ++nu) row[nu] = rows.v[mu * n + nu];
      a[c * n + mu] = face_dot<T>(row, [&](int nu) { return v[c * n + nu]; });
    }
}
template <typename T>
__device__ __forceinline__ Sides<T> zline_sides(const Tab<K, T>* __restrict__ t, const T* ext,
                                                int N, const PatchPos& P, int px, int py) {
  Sides<T> sd = bare_sides<T>(P.lo[2], N, false);
  const T* z = ext + 4 * NF;
  if (!sd.bl) { sd.aL = ext_my<T>(t, z + 0 * NF, px, py); sd.bL = ext_my<T>(t, z + 1 * NF, px, py); }
  if (!sd.br) { sd.aR = ext_my<T>(t, z + 2 * NF, px, py); sd.bR = ext_my<T>(t, z + 3 * NF, px, py); }
  return sd;
}

// Read x-line (py, pz) from global.
template <typename T>
__device__ __forceinline__ void read_xline(const T* __restrict__ x, long long row0, Line<T>& v) {
#pragma unroll
  for (int a = 0; a < n; ++a) {
    v.v[a] = x[row0 + a];
    v.v[n + a] = x[row0 + NC + a];
  }
}

// Lines of a patch within one wave (3-D Q1, Q3: TPP = 16 or 64 lanes): values
// held one per lane can be contracted across lanes.
constexpr bool kZShfl = (TPP <= 64) && (64 % TPP == 0);

// sum_nu row[nu] v(lane + LQ (nu - mu)): the y-contraction of z-face values
// held one per lane (wl: the lane's index in its wave; LQ: lanes between nodes
// consecutive in y)
template <typename T, int LQ = E>
__device__ __forceinline__ T ycontract_lanes(const T (&row)[n], T v, int wl, int mu) {
  return face_dot<T>(row, [&](int nu) { return __shfl(v, wl + LQ * (nu - mu), 64); });
}

// Couplings (alpha, beta) of one face node of a neighbour cell across a y-
// or z-face from the node's n values along the normal, v[j] (SIDE 0: the
// neighbour below, read at its far end; SIDE 1: above, read at its near end).
template <typename T, int SIDE>
__device__ __forceinline__ void face_node(T sg, const T (&v)[n], T& al, T& be) {
  const T half = T(0.5);
  const T tr = v[SIDE == 0 ? K : 0];
  al = face_alpha<T, SIDE>(sg, face_grad<T, SIDE>([&](int j) { return v[j]; }), tr);
  be = (SIDE == 0) ? -half * tr : half * tr;
}

// The lanes of an x-block (n consecutive lanes of a row of E) are one quad or
// half of one where n is 4 or 2 (Q1, Q3).
constexpr bool kFaceDPP = (n == 2 || n == 4);

// sum_nu row[nu] v(lane of node nu in this lane's x-block): the mass
// contraction of per-node face values held one per lane; every lane of the
// block takes part
// Node NU of this lane's x-block, read by a DPP quad permutation (x-blocks of
// 2 or 4 lanes lie in one quad): a VALU move per 32 bits, no LDS crossbar.
template <int NU>
__device__ __forceinline__ constexpr int xblock_dpp() {
  return (n == 4) ? NU * 0x55 : (NU | (NU << 2) | ((2 + NU) << 4) | ((2 + NU) << 6));
}
template <int CTRL>
__device__ __forceinline__ double dpp_bcast(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <typename T>
__device__ __forceinline__ T xcontract_lanes(const T (&row)[n], T v) {
  T s = T(0);
  if constexpr (kFaceDPP) {
    s += row[0] * dpp_bcast<xblock_dpp<0>()>(v);
    s += row[1] * dpp_bcast<xblock_dpp<1>()>(v);
    if constexpr (n == 4) {
      s += row[2] * dpp_bcast<xblock_dpp<2>()>(v);
      s += row[3] * dpp_bcast<xblock_dpp<3>()>(v);
    }
  }
  return s;
}

// Dirichlet smoothers' z-face traces in registers (patches of one wave): lane
// (px, py) holds the traces of its x-block on each z-neighbour contracted with
// its mass row (operator_passes), and the z-line (px, py = lane / E) contracts
// them along y across lanes; rowy: the mass row of py
template <typename T>
__device__ __forceinline__ Sides<T> rfz_sides(const T (&rowy)[n], int N, const PatchPos& P, int lane, T wz0, T wz1) {
  Sides<T> sd = bare_sides<T>(P.lo[2], N, false);
  const int py = lane / E;
  const int wl = threadIdx.x & 63;
  const T zL = ycontract_lanes<T>(rowy, wz0, wl, py % n);
  const T zR = ycontract_lanes<T>(rowy, wz1, wl, py % n);
  if (!sd.bl) sd.bL = zL;
  if (!sd.br) sd.bR = zR;
  return sd;
}

// Operator passes of y = A_ref x on the patch.  Phase X0 reads the x-lines
// from global (and keeps them in xl for the caller), gathers the y/z face
// data; the last pass (z in 3-D, y in 2-D) hands each output line to
// emit(line, base, stride, y).  A, B: LDS tiles; ext: LDS face data.
// RFA (operator data, patches of one wave): the y- and z-neighbour face data
// in registers and across lanes as in k_apply_rf instead of the LDS arrays.
template <typename T, int MODE, bool RFA = false, typename Emit>
__device__ __forceinline__ void operator_passes(const Tab<K, T>* __restrict__ t, const T* __restrict__ x,
                                                int N, const PatchPos& P, T* A, T* B, T* ext,
                                                int lane, bool active, Line<T>& xl, Emit emit) {
  // The Dirichlet residual with z-face traces (3-D Q1, a patch within a wave): these go
  // through registers.  Lane (px, py) reads the n traces of its x-block on each
  // z-neighbour and contracts beta = -+t/2 with its mass row, the Z pass contracts
  // along y across lanes.
  constexpr bool RFZ = (D == 3) && MODE == 1;
  static_assert(!RFZ || kZShfl, "patches of several waves take the direct form");
  static_assert(!RFA || (MODE == 0 && D == 3 && kZShfl), "register face data: 3-D operator, one wave");
  T wz0 = T(0), wz1 = T(0);
  T ya0 = T(0), yb0 = T(0), ya1 = T(0), yb1 = T(0);  // RFA: y-line (px, pz) = (lane % E, lane / E)
  T za0 = T(0), zb0 = T(0), za1 = T(0), zb1 = T(0);  // RFA: z-face node (px, py) = (lane % E, lane / E)
  // the smoothers' residual is only used on V_j: along each direction the two
  // tile ends are skipped unless they lie on the domain boundary (outputs left
  // at the ends are never read by a used result)
  const bool n0x = MODE == 0 || (P.ty[0] & 1), nEx = MODE == 0 || (P.ty[0] & 2);
  const bool n0y = MODE == 0 || (P.ty[1] & 1), nEy = MODE == 0 || (P.ty[1] & 2);
  const bool n0z = MODE == 0 || (P.ty[2] & 1), nEz = MODE == 0 || (P.ty[2] & 2);
  // smoothers: y-face sides of the lane's y-line straight from global, and
  // (RFZ) the mass row of the z-line's py for the Z pass
  Sides<T> ysd_global{};
  T rowz[n];
  // X0: a = M_x x -> A, b = L_x x -> B
  if (MODE != 0 && active) {
    // Smoothers: every global load of the pass is
    // issued before any of the values is used (one memory round trip instead
    // of one per helper), then the arithmetic
    const int px = lane % E, q = lane / E;  // y-line (px, pz = q), z-face node (px, py = q)
    YSideRaw<T> yraw;
    yside_load<T, MODE>(x, N, P, px, (D == 3) ? q : 0, yraw);
    T zl[n], zr[n];
    if constexpr (RFZ) {
      const int cx = P.lo[0] + px / n, cy = P.lo[1] + q / n;
      const long long o = (long long)n * (q % n);
      const T* cl = x + cell_index(N, cx, cy, P.lo[2] > 0 ? P.lo[2] - 1 : P.lo[2]) * NC + o + K * n * n;
      const T* cr = x + cell_index(N, cx, cy, P.lo[2] + 2 < N ? P.lo[2] + 2 : P.lo[2]) * NC + o;
#pragma unroll
      for (int nu = 0; nu < n; ++nu) {
        zl[nu] = cl[nu];
        zr[nu] = cr[nu];
      }
      face_row<T>(q % n, rowz);
    }
    const int py = lane % E, pz = lane / E;
    const long long row0 = xrow_offset(N, P, py, pz);
    read_xline<T>(x, row0, xl);
    const bool xbl = (P.lo[0] == 0), xbr = (P.lo[0] + 1 == N - 1);
    T xtl = T(0), xtr = T(0);
    if (MODE != 2) {
      xtl = x[xbl ? row0 : row0 - NC + K];
      xtr = x[xbr ? row0 : row0 + 2 * NC];
    }
    ysd_global = yside_finish<T, MODE>(yraw, N, P);
    if constexpr (RFZ) {
      const T half = T(0.5);
      if (P.lo[2] > 0) {
        T s = T(0);
#pragma unroll
        for (int nu = 0; nu < n; ++nu) s += yraw.row[nu] * (-half * zl[nu]);
        wz0 = s;
      }
      if (P.lo[2] + 2 < N) {
        T s = T(0);
#pragma unroll
        for (int nu = 0; nu < n; ++nu) s += yraw.row[nu] * (half * zr[nu]);
        wz1 = s;
      }
    }
    Sides<T> sd = bare_sides<T>(P.lo[0], N, MODE == 2);
    if (MODE != 2) {
      if (!sd.bl) sd.bL = -T(0.5) * xtl;
      if (!sd.br) sd.bR = T(0.5) * xtr;
    }
    int base, stride;
    line_geom(0, lane, base, stride);
    Line<T> a, b;
    line_mass<T>(t, xl, a, n0x, nEx);
    line_sipg<T, false>(t, xl, sd, b, n0x, nEx);
    store_line(A, base, stride, a);
    store_line(B, base, stride, b);
  } else if (RFA && active) {
    static_assert(!RFA || kFaceDPP, "x-blocks within a quad");
    // register face data (operator, patches of one wave): every global load
    // first, as in k_apply_rf -- this lane's node column of each neighbour
    // face block, the x-line and its x-neighbours' rows -- then the per-node
    // face couplings, contracted with M_x across the lanes of the x-block
    const int px = lane % E, q = lane / E, nuo = px % n;
    const int wl = threadIdx.x & 63;
    const int cx = P.lo[0] + px / n;
    const bool ybl = (P.lo[1] == 0), ybr = (P.lo[1] + 1 == N - 1);
    const bool zbl = (P.lo[2] == 0), zbr = (P.lo[2] + 1 == N - 1);
    T fy0[n], fy1[n], fz0[n], fz1[n];
    {
      const int cz = P.lo[2] + q / n;
      const long long o = (long long)(n * n) * (q % n) + nuo;
      const T* c0 = x + cell_index(N, cx, ybl ? P.lo[1] : P.lo[1] - 1, cz) * NC + o;
      const T* c1 = x + cell_index(N, cx, ybr ? P.lo[1] + 1 : P.lo[1] + 2, cz) * NC + o;
#pragma unroll
      for (int j = 0; j < n; ++j) {
        fy0[j] = c0[j * n];
        fy1[j] = c1[j * n];
      }
    }
    {
      const int cy = P.lo[1] + q / n;
      const long long o = (long long)n * (q % n) + nuo;
      const T* c0 = x + cell_index(N, cx, cy, zbl ? P.lo[2] : P.lo[2] - 1) * NC + o;
      const T* c1 = x + cell_index(N, cx, cy, zbr ? P.lo[2] + 1 : P.lo[2] + 2) * NC + o;
#pragma unroll
      for (int j = 0; j < n; ++j) {
        fz0[j] = c0[j * n * n];
        fz1[j] = c1[j * n * n];
      }
    }
    const int py = lane % E, pz = lane / E;
    const long long row0 = xrow_offset(N, P, py, pz);
    read_xline<T>(x, row0, xl);
    const bool xbl = (P.lo[0] == 0), xbr = (P.lo[0] + 1 == N - 1);
    T rl[n], rr[n];
    {
      const T* r0 = x + (xbl ? row0 : row0 - NC);
      const T* r1 = x + (xbr ? row0 : row0 + 2 * NC);
#pragma unroll
      for (int j = 0; j < n; ++j) {
        rl[j] = r0[j];
        rr[j] = r1[j];
      }
    }
    T rowx[n];
    face_row<T>(nuo, rowx);
    face_row<T>(q % n, rowz);
    const T sg = t->sigma;
    T nya0, nyb0, nya1, nyb1, nza0, nzb0, nza1, nzb1;
    face_node<T, 0>(sg, fy0, nya0, nyb0);
    face_node<T, 1>(sg, fy1, nya1, nyb1);
    face_node<T, 0>(sg, fz0, nza0, nzb0);
    face_node<T, 1>(sg, fz1, nza1, nzb1);
    const Sides<T> sd = xsides_rows<T>(sg, xbl, xbr, rl, rr);
    int base, stride;
    line_geom(0, lane, base, stride);
    Line<T> a, b;
    line_mass<T>(t, xl, a, n0x, nEx);
    line_sipg<T, false>(t, xl, sd, b, n0x, nEx);
    store_line(A, base, stride, a);
    store_line(B, base, stride, b);
    const T sya0 = xcontract_lanes<T>(rowx, nya0), syb0 = xcontract_lanes<T>(rowx, nyb0);
    const T sya1 = xcontract_lanes<T>(rowx, nya1), syb1 = xcontract_lanes<T>(rowx, nyb1);
    const T sza0 = xcontract_lanes<T>(rowx, nza0), szb0 = xcontract_lanes<T>(rowx, nzb0);
    const T sza1 = xcontract_lanes<T>(rowx, nza1), szb1 = xcontract_lanes<T>(rowx, nzb1);
    if (!ybl) { ya0 = sya0; yb0 = syb0; }
    if (!ybr) { ya1 = sya1; yb1 = syb1; }
    if (!zbl) { za0 = sza0; zb0 = szb0; }
    if (!zbr) { za1 = sza1; zb1 = szb1; }
  } else if (active) {
    gather_ext<T>(t, x, N, P, lane, ext);
    const long long row0 = xrow_offset(N, P, lane % E, lane / E);
    read_xline<T>(x, row0, xl);
    const Sides<T> sd = xline_sides<T>(t, x, N, P, row0);
    int base, stride;
    line_geom(0, lane, base, stride);
    Line<T> a, b;
    line_mass<T>(t, xl, a, n0x, nEx);
    line_sipg<T, false>(t, xl, sd, b, n0x, nEx);
    store_line(A, base, stride, a);
    store_line(B, base, stride, b);
  }
  __syncthreads();
  if constexpr (D == 3) {
    // Y: c = M_y b + L_y a -> B, d = M_y a -> A; z-face data contracted along x
    if (active) {
      // one y-line per lane, then, for face data in LDS, lanes 0 .. 4 E - 1
      // contract one z-face row each along x (the y-lines read only the y-face
      // arrays of ext)
      {
        const int i = lane;
        {
          const int px = i % E, pz = i / E;
          int base, stride;
          line_geom(1, i, base, stride);
          Line<T> a, b, c, d;
          load_line(A, base, stride, a);
          load_line(B, base, stride, b);
          Sides<T> sd;
          if constexpr (RFA) {
            sd.bl = (P.lo[1] == 0);
            sd.br = (P.lo[1] + 1 == N - 1);
            sd.aL = ya0;
            sd.bL = yb0;
            sd.aR = ya1;
            sd.bR = yb1;
            sd.lit = false;
          } else {
            sd = (MODE == 0) ? yline_sides<T>(t, ext, N, P, px, pz) : ysd_global;
          }
          line_mass<T>(t, b, c, n0y, nEy);
          line_sipg<T, true>(t, a, sd, c, n0y, nEy);
          line_mass<T>(t, a, d, n0y, nEy);
          store_line(B, base, stride, c);
          store_line(A, base, stride, d);
        }
      }
      if constexpr (MODE == 0 && !RFA)
        if (lane < 4 * E) extz_mass_x_line<T>(t, ext, lane);
    }
    __syncthreads();
    // Z: y = M_z c + L_z d
    if (active) {
      for (int i = lane; i < NL; i += TPP) {
        const int px = i % E, py = i / E;
        int base, stride;
        line_geom(2, i, base, stride);
        Line<T> c, d, y;
        load_line(B, base, stride, c);
        load_line(A, base, stride, d);
        Sides<T> sd;
        if constexpr (RFZ) {
          sd = rfz_sides<T>(rowz, N, P, i, wz0, wz1);
        } else if constexpr (MODE == 2) {
          sd = bare_sides<T>(P.lo[2], N, true);
        } else if constexpr (RFA) {
          const int wl = threadIdx.x & 63;
          const T zaL = ycontract_lanes<T>(rowz, za0, wl, py % n);
          const T zbL = ycontract_lanes<T>(rowz, zb0, wl, py % n);
          const T zaR = ycontract_lanes<T>(rowz, za1, wl, py % n);
          const T zbR = ycontract_lanes<T>(rowz, zb1, wl, py % n);
          sd.bl = (P.lo[2] == 0);
          sd.br = (P.lo[2] + 1 == N - 1);
          sd.aL = sd.bl ? T(0) : zaL;
          sd.bL = sd.bl ? T(0) : zbL;
          sd.aR = sd.br ? T(0) : zaR;
          sd.bR = sd.br ? T(0) : zbR;
          sd.lit = false;
        } else {
          sd = zline_sides<T>(t, ext, N, P, px, py);
        }
        line_mass<T>(t, c, y, n0z, nEz);
        line_sipg<T, true>(t, d, sd, y, n0z, nEz);
        emit(i, base, stride, y);
      }
    }
  } else {
    // Y (2-D): y = M_y b + L_y a
    if (active) {
      for (int i = lane; i < NL; i += TPP) {
        const int px = i;
        int base, stride;
        line_geom(1, i, base, stride);
        Line<T> a, b, y;
        load_line(A, base, stride, a);
        load_line(B, base, stride, b);
        const Sides<T> sd = (MODE == 0) ? yline_sides<T>(t, ext, N, P, px, 0) : ysd_global;
        line_mass<T>(t, b, y, n0y, nEy);
        line_sipg<T, true>(t, a, sd, y, n0y, nEy);
        emit(i, base, stride, y);
      }
    }
  }
}

// Load the last-direction line of b (z-line in 3-D, y-line in 2-D) at line l.
template <typename T>
__device__ __forceinline__ void read_lastline(const T* __restrict__ b, int N, const PatchPos& P, int l,
                                              Line<T>& v) {
  if constexpr (D == 3) {
    const long long base = node_offset(N, P, l % E, l / E, 0);
    const long long cz = (long long)N * N * NC;  // next cell in z
#pragma unroll
    for (int p = 0; p < E; ++p) v.v[p] = b[base + (p / n) * cz + (p % n) * (n * n)];
  } else {
    const long long base = node_offset(N, P, l, 0, 0);
    const long long cy = (long long)N * NC;      // next cell in y
#pragma unroll
    for (int p = 0; p < E; ++p) v.v[p] = b[base + (p / n) * cy + (p % n) * n];
  }
}

template <int NB, int NEXTV>
struct Smem {
  static constexpr int per_patch = NB * TS + NEXTV;
};

// ---------------------------------------------------------------- apply
template <typename T, int PPB, bool RP = false>
__global__ void __launch_bounds__(TPP * PPB)
k_apply(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, const T* __restrict__ x,
        T* __restrict__ y, long long ndof) {
  constexpr int PP = Smem<2, (D - 1) * 2 * 2 * NF>::per_patch;
  __shared__ T smem[PPB * PP];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  int pid, rhs;
  slot_work<PPB, RP>(g, slot, pid, rhs);
  const bool active = pid < g.npatch;
  T* A = smem + slot * PP;
  T* B = A + TS;
  T* ext = B + TS;
  const long long roff = (long long)rhs * ndof;
  const T* xr = x + roff;
  T* yr = y + roff;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  Line<T> xl;
  operator_passes<T, 0>(t, xr, g.N, P, A, B, ext, lane, active, xl,
                        [&](int, int base, int stride, const Line<T>& v) {
#pragma unroll
                          for (int p = 0; p < E; ++p) A[base + p * stride] = scale * v.v[p];
                        });
  __syncthreads();
  // X2: contiguous row stores
  if (active) {
    for (int i = lane; i < NL; i += TPP) {
      const int py = i % E, pz = i / E;
      int base, stride;
      line_geom(0, i, base, stride);
      const long long row0 = xrow_offset(g.N, P, py, pz);
#pragma unroll
      for (int a = 0; a < n; ++a) {
        yr[row0 + a] = A[base + a];
        yr[row0 + NC + a] = A[base + n + a];
      }
    }
  }
}

// ------------------------------------------- apply, face data in registers
// Each lane forms the couplings alpha, beta of one node of each y- and z-face
// from its own node column of the neighbour (n values along the normal), and
// the mass contractions along x and y run across lanes where a patch's lines
// sit in one wave (Q1, Q3: TPP = 16 or 64 lanes), otherwise through LDS (12
// values a face node, in the space the tiles take afterwards).  The sums are
// those of gather_ext / ext_mx / extz_mass_x_line / ext_my in the same order,
// so the result equals k_apply bit for bit.
// What bounds it: memory requests, then wavefronts in flight.  The lanes run
// through a plane cell by cell and the z-lines go straight from registers to
// memory, n^2 consecutive values a cell: written row by row from a tile, a
// wave's 16-byte pieces cost four times the write requests of the values (Q7
// FP64: 512 a wave instead of 128) and a phase more.  Measured on 32^3 cells,
// x-rows out / z-lines out: Q4 x 16 right-hand sides FP64 394 / 356 us, FP32 234 /
// 211 us; Q6 79 / 76 us; Q7 113 / 98 us.
// One tile where two leave fewer than four patches of four waves a CU (Q7 in
// FP64: 70 KB): M_x x goes through it to the y-lines, then L_x x, likewise the
// two y-results; two barriers more each, three patches a CU instead of two: 98 /
// 91 us (64^3: 839 us on two tiles with x-rows out, 711 us now, 3.0 TB/s of
// the 2.1 GB it reads and writes).  For the other degrees one tile measured the same or up to 2%
// slower.
constexpr bool kApplyRF = (D == 3);
template <typename T>
constexpr bool kApplyOne = 2 * TS * (int)sizeof(T) > 64 * 1024;
template <typename T>
constexpr int kApplyTiles = kApplyOne<T> ? TS : 2 * TS;
template <typename T>
constexpr int kApplyRFPP = kZShfl || kApplyTiles<T> > 12 * NF ? kApplyTiles<T> : 12 * NF;

template <typename T>
__device__ __forceinline__ void restrict_tail(const PatchGrid& g, const PatchPos& P, T* A, T* __restrict__ bc,
                                              long long ndof_c, int rhs, int lane, bool active);

// One patch of the register-face operator (pid, right-hand side rhs; lane =
// thread within the patch, A = its LDS, active: the patch takes part; xl
// returns the lane's x-line of x).  What follows the operator's last pass:
//   RF_APPLY: y = scale A x on the patch cells;
//   RF_RESTRICT: the residual restriction of k_restrict, bc = P^T (b - scale
//     A x) into the patch's coarse cell (y is bc there), with the same values
//     (the operator output and the P^T contractions in the same order);
//   RF_EMIT: emit(l, base, stride, v) with the operator output v of z-line l
//     (as operator_passes hands it to the Full smoother), nothing after it.
// All on the smaller LDS footprint of this kernel (kApplyRFPP).
constexpr int RF_APPLY = 0, RF_RESTRICT = 1, RF_EMIT = 2;
template <typename T, int OUT, typename Emit = int>
__device__ __forceinline__ void apply_rf_body(const Tab<K, T>* t, const PatchGrid& g, T scale, const T* x, T* y,
                                              const T* b, long long ndof, long long ndof_c, int pid, int lane,
                                              T* A, int rhs, bool active, Line<T>& xl, Emit emit = 0) {
  // cross-lane reads stay within a patch's lanes, which lie in one wave
  static_assert(kApplyRF, "3-D only");
  const int wl = threadIdx.x & 63;
  T* B = kApplyOne<T> ? A : A + TS;
  const long long roff = (long long)rhs * ndof;
  const T* xr = x + roff;
  const int N = g.N;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  // this lane's lines: x (py = px, pz = q), y (px, pz = q), z (px, py = q) and
  // its face nodes of the same numbers; the lanes run through a plane cell by
  // cell (RF_EMIT: row by row, the order of its caller's lines)
  constexpr bool CM = OUT != RF_EMIT;
  constexpr int LQ = CM ? n : E;  // lanes from one q to the next within a cell
  const int px = CM ? (lane / (n * n)) % 2 * n + lane % n : lane % E;
  const int q = CM ? lane / (2 * n * n) * n + lane / n % n : lane / E;
  const int ln = px + E * q;
  T rowx[n], rowy[n];
  face_row<T>(px % n, rowx);
  if constexpr (kFaceDPP) face_row<T>(q % n, rowy);
  const bool ybl = (P.lo[1] == 0), ybr = (P.lo[1] + 1 == N - 1);
  const bool zbl = (P.lo[2] == 0), zbr = (P.lo[2] + 1 == N - 1);
  T ya0 = T(0), yb0 = T(0), ya1 = T(0), yb1 = T(0);
  T za0 = T(0), zb0 = T(0), za1 = T(0), zb1 = T(0);
  // per-node face couplings of this lane's node nuo of its x-block
  T nya0 = T(0), nyb0 = T(0), nya1 = T(0), nyb1 = T(0);
  T nza0 = T(0), nzb0 = T(0), nza1 = T(0), nzb1 = T(0);
  const int nuo = px % n;
  Sides<T> xsd{};
  if (active) {
    // Every global load first (one memory round trip): this lane's node
    // column of each neighbour face block (n values along the normal), the
    // x-line and the rows of its x-neighbours; missing neighbours read the
    // patch's own cells, whose values go unused.
    const int cx = P.lo[0] + px / n;
    T fy0[n], fy1[n], fz0[n], fz1[n];
    {
      const int cz = P.lo[2] + q / n;
      const long long o = (long long)(n * n) * (q % n) + nuo;
      const T* c0 = xr + cell_index(N, cx, ybl ? P.lo[1] : P.lo[1] - 1, cz) * NC + o;
      const T* c1 = xr + cell_index(N, cx, ybr ? P.lo[1] + 1 : P.lo[1] + 2, cz) * NC + o;
#pragma unroll
      for (int j = 0; j < n; ++j) {
        fy0[j] = c0[j * n];
        fy1[j] = c1[j * n];
      }
    }
    {
      const int cy = P.lo[1] + q / n;
      const long long o = (long long)n * (q % n) + nuo;
      const T* c0 = xr + cell_index(N, cx, cy, zbl ? P.lo[2] : P.lo[2] - 1) * NC + o;
      const T* c1 = xr + cell_index(N, cx, cy, zbr ? P.lo[2] + 1 : P.lo[2] + 2) * NC + o;
#pragma unroll
      for (int j = 0; j < n; ++j) {
        fz0[j] = c0[j * n * n];
        fz1[j] = c1[j * n * n];
      }
    }
    const long long row0 = xrow_offset(N, P, px, q);
    read_xline<T>(xr, row0, xl);
    const bool xbl = (P.lo[0] == 0), xbr = (P.lo[0] + 1 == N - 1);
    T rl[n], rr[n];
    {
      const T* r0 = xr + (xbl ? row0 : row0 - NC);
      const T* r1 = xr + (xbr ? row0 : row0 + 2 * NC);
#pragma unroll
      for (int j = 0; j < n; ++j) {
        rl[j] = r0[j];
        rr[j] = r1[j];
      }
    }
    const T sg = t->sigma;
    face_node<T, 0>(sg, fy0, nya0, nyb0);
    face_node<T, 1>(sg, fy1, nya1, nyb1);
    face_node<T, 0>(sg, fz0, nza0, nzb0);
    face_node<T, 1>(sg, fz1, nza1, nzb1);
    xsd = xsides_rows<T>(sg, xbl, xbr, rl, rr);
    if constexpr (!kFaceDPP) {
      // node couplings to LDS, in the space the tiles take afterwards
      const T nv[8] = {nya0, nyb0, nya1, nyb1, nza0, nzb0, nza1, nzb1};
#pragma unroll
      for (int f = 0; f < 8; ++f) A[f * NF + lane] = nv[f];
    }
  }
  // face couplings contracted with M_x over the nodes of each x-block: across
  // lanes by DPP where a block is a quad or less (Q1, Q3), else from LDS.  (All
  // lanes of a patch take part.)
  T fc[8];
  if constexpr (kFaceDPP) {
    fc[0] = xcontract_lanes<T>(rowx, nya0), fc[1] = xcontract_lanes<T>(rowx, nyb0);
    fc[2] = xcontract_lanes<T>(rowx, nya1), fc[3] = xcontract_lanes<T>(rowx, nyb1);
    fc[4] = xcontract_lanes<T>(rowx, nza0), fc[5] = xcontract_lanes<T>(rowx, nzb0);
    fc[6] = xcontract_lanes<T>(rowx, nza1), fc[7] = xcontract_lanes<T>(rowx, nzb1);
  } else {
    __syncthreads();
    // (read only now: with the first loads they cost Q7 in FP64 its third wave)
    face_row<T>(q % n, rowy);
    if (active) {
      const T* w = A + lane - nuo;
#pragma unroll
      for (int f = 0; f < 8; ++f) fc[f] = face_dot<T>(rowx, [&](int nu) { return w[f * NF + nu]; });
    }
  }
  if (active) {
    if (!ybl) { ya0 = fc[0]; yb0 = fc[1]; }
    if (!ybr) { ya1 = fc[2]; yb1 = fc[3]; }
    if (!zbl) { za0 = fc[4]; zb0 = fc[5]; }
    if (!zbr) { za1 = fc[6]; zb1 = fc[7]; }
  }
  const int muy = q % n;
  T zaL = T(0), zbL = T(0), zaR = T(0), zbR = T(0);
  if constexpr (kZShfl) {  // (all lanes of a patch take part)
    zaL = ycontract_lanes<T, LQ>(rowy, za0, wl, muy);
    zbL = ycontract_lanes<T, LQ>(rowy, zb0, wl, muy);
    zaR = ycontract_lanes<T, LQ>(rowy, za1, wl, muy);
    zbR = ycontract_lanes<T, LQ>(rowy, zb1, wl, muy);
  } else {
    T* wz = A + 8 * NF;  // beyond the node couplings, which may still be read
    if (active) {
      wz[0 * NF + lane] = za0;
      wz[1 * NF + lane] = zb0;
      wz[2 * NF + lane] = za1;
      wz[3 * NF + lane] = zb1;
    }
    __syncthreads();
    if (active) {
      const int f0 = lane - LQ * muy;
      auto zrow = [&](int f) { return face_dot<T>(rowy, [&](int nu) { return wz[f * NF + f0 + LQ * nu]; }); };
      zaL = zrow(0);
      zbL = zrow(1);
      zaR = zrow(2);
      zbR = zrow(3);
    }
    __syncthreads();
  }
  int bx, sx, by, sy, base, stride;
  line_geom(0, ln, bx, sx);
  line_geom(1, ln, by, sy);
  line_geom(2, ln, base, stride);
  Line<T> la, lb, lc, ld, o;
  // X: a = M_x x, b = L_x x
  if (active) {
    line_mass<T>(t, xl, la);
    line_sipg<T, false>(t, xl, xsd, lb);
    store_line(A, bx, sx, la);
    if constexpr (!kApplyOne<T>) store_line(B, bx, sx, lb);
  }
  __syncthreads();
  // Y: c = M_y b + L_y la, d = M_y a
  if (active) load_line(A, by, sy, la);
  if constexpr (kApplyOne<T>) {
    __syncthreads();
    if (active) store_line(A, bx, sx, lb);
    __syncthreads();
  }
  if (active) {
    load_line(B, by, sy, lb);
    Sides<T> sd;
    sd.bl = ybl;
    sd.br = ybr;
    sd.aL = ya0;
    sd.bL = yb0;
    sd.aR = ya1;
    sd.bR = yb1;
    sd.lit = false;
    line_mass<T>(t, lb, lc);
    line_sipg<T, true>(t, la, sd, lc);
    line_mass<T>(t, la, ld);
    store_line(B, by, sy, lc);
    if constexpr (!kApplyOne<T>) store_line(A, by, sy, ld);
  }
  __syncthreads();
  // Z: y = M_z c + L_z d
  if (active) load_line(B, base, stride, lc);
  if constexpr (kApplyOne<T>) {
    __syncthreads();
    if (active) store_line(A, by, sy, ld);
    __syncthreads();
  }
  if (active) {
    load_line(A, base, stride, ld);
    Sides<T> sd;
    sd.bl = zbl;
    sd.br = zbr;
    sd.aL = zbl ? T(0) : zaL;
    sd.bL = zbl ? T(0) : zbL;
    sd.aR = zbr ? T(0) : zaR;
    sd.bR = zbr ? T(0) : zbR;
    sd.lit = false;
    line_mass<T>(t, lc, o);
    line_sipg<T, true>(t, ld, sd, o);
    if constexpr (OUT == RF_EMIT) {
      emit(ln, base, stride, o);
    } else if constexpr (OUT == RF_RESTRICT) {
      // r = b - scale A x on this z-line, contracted with P^T along z
      Line<T> r;
      read_lastline<T>(b + roff, N, P, ln, r);
#pragma unroll
      for (int nu = 0; nu < n; ++nu) {
        T s = T(0);
#pragma unroll
        for (int p = 0; p < E; ++p) s += T(kRef.P[p * n + nu]) * (r.v[p] - scale * o.v[p]);
        A[base + nu * stride] = s;
      }
    } else {
      // straight to memory: the lanes of a cell write n^2 consecutive values
      T* yz = y + roff + node_offset(N, P, px, q, 0);
      const long long cz = (long long)N * N * NC;
#pragma unroll
      for (int p = 0; p < E; ++p) yz[(p / n) * cz + (p % n) * (n * n)] = scale * o.v[p];
    }
  }
  if constexpr (OUT == RF_RESTRICT) {
    __syncthreads();
    restrict_tail<T>(g, P, A, y, ndof_c, rhs, lane, active);
  }
}

template <typename T, int PPB, bool RP = false>
__global__ void __launch_bounds__(TPP * PPB)
k_apply_rf(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, const T* __restrict__ x,
           T* __restrict__ y, long long ndof) {
  __shared__ T smem[PPB * kApplyRFPP<T>];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  int pid, rhs;
  slot_work<PPB, RP>(g, slot, pid, rhs);
  Line<T> xl;
  apply_rf_body<T, RF_APPLY>(t, g, scale, x, y, nullptr, ndof, 0, pid, lane, smem + slot * kApplyRFPP<T>, rhs,
                             pid < g.npatch, xl);
}

// ----------------------------------------------------------------- mass
template <typename T, int PPB>
__global__ void __launch_bounds__(TPP * PPB)
k_mass(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, const T* __restrict__ x,
       T* __restrict__ y, long long ndof) {
  __shared__ T smem[PPB * TS];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  const int pid = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap) * PPB + slot;
  const bool active = pid < g.npatch;
  T* tile = smem + slot * TS;
  const long long roff = (long long)blockIdx.y * ndof;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  if (active) {
    for (int i = lane; i < NL; i += TPP) {
      const int py = i % E, pz = i / E;
      int base, stride;
      line_geom(0, i, base, stride);
      Line<T> v, o;
      read_xline<T>(x + roff, xrow_offset(g.N, P, py, pz), v);
      line_mass<T>(t, v, o);
      store_line(tile, base, stride, o);
    }
  }
  __syncthreads();
#pragma unroll
  for (int dir = 1; dir < D; ++dir) {
    if (active) {
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(dir, i, base, stride);
        Line<T> v, o;
        load_line(tile, base, stride, v);
        line_mass<T>(t, v, o);
        store_line(tile, base, stride, o);
      }
    }
    __syncthreads();
  }
  if (active) {
    for (int i = lane; i < NL; i += TPP) {
      const int py = i % E, pz = i / E;
      int base, stride;
      line_geom(0, i, base, stride);
      const long long row0 = xrow_offset(g.N, P, py, pz);
#pragma unroll
      for (int a = 0; a < n; ++a) {
        y[roff + row0 + a] = scale * tile[base + a];
        y[roff + row0 + NC + a] = scale * tile[base + n + a];
      }
    }
  }
}

// -------------------------------------------------------------- smoother
// One colour of Alg. 1: local residual on the patch, then fast
// diagonalisation x|V_j += (x)S (sum lambda)^{-1} (x)S^T r_j.
//   MODE 1: Dirichlet kernel, consistent residual (b - A x)|V_j, in place;
//   MODE 2: Dirichlet kernel, the paper's residual: patch cells only, the
//           consistency term left out on interior outer faces; in place;
//   MODE 3: Full kernel: V_j = the whole patch, r = (b - A x)|patch with x taken
//           from xin, result written to xout.  Same-colour patches read each
//           other's cells (face neighbours), so the colour reads one copy of x
//           and writes the other; the launch also carries the partial patches
//           at the mesh boundary, which copy their in-domain cells unchanged.
//   MODE 4: clamped kernel: the residual from the patch cells alone (the
//           terms it misses act on directions the clamped space annihilates),
//           the FD solve on the clamped space; in place.
// ZERO: x = 0 on entry and the launch is colour 0, whose patches tile the mesh:
// the residual is b itself (no operator pass, x is not read) and every tile
// row is written (zeros outside V_j), so x needs no clearing beforehand.
// LDS per patch of the smoother: operator face data (full rows) for the Full
// kernel, z-face traces only for the Dirichlet and clamped kernels
// The Full kernel's operator pass takes the neighbour face data in registers
// in 3-D, as the apply and the restriction do: on patches within one wave (Q1,
// Q3) through operator_passes (two tiles of LDS per patch), otherwise through
// the apply's register-face body (kApplyRFPP of LDS per patch); no face
// arrays either way.
constexpr bool kFullRF = (D == 3) && kZShfl;
constexpr bool kFullOnApplyRF = kApplyRF && !kFullRF;
// The Dirichlet smoothers (MODE 1, 2) take the direct form (gs_body) where
// direct_smoother says so.
template <int MODE>
constexpr bool kDirect = (MODE == 1 || MODE == 2) && direct_smoother(D, K);
// MODE 5, 6: MODE 1, 2 by operator passes, on the levels where direct_below has the
// direct form give way
template <typename T>
constexpr bool kBothForms = direct_smoother(D, K) && direct_below(D, K, sizeof(T)) != kAllLevels;

// LDS of the direct form per patch: the tile, whose space first holds the face
// fields -- in 3-D 16 planes of E x E values with the tile's row and plane
// strides (so that lines along either direction of a plane are read without
// bank conflicts), in 2-D 8 rows of E.
// In 3-D the mass matrix follows where n > 4.
constexpr int kGsM = (16 > E ? 16 : E) * SZ;
constexpr int kGsPP = (D == 3) ? kGsM + (n > 4 ? n * n : 0) : (TS > 8 * E ? TS : 8 * E);
template <int MODE, typename T = double>
__host__ __device__ constexpr int smooth_pp() {
  return kDirect<MODE> ? kGsPP
         : MODE == 3 ? (kFullRF ? 2 * TS : kFullOnApplyRF ? kApplyRFPP<T> : Smem<2, (D - 1) * 2 * 2 * NF>::per_patch)
                   : 2 * TS;
}

// ------------------------------------- Dirichlet smoothers, direct form
// A Dirichlet patch's update x_V + A_VV^{-1} (b - A x)_V does not depend on the
// old values on V: it is the solution of A_VV x_V = b_V - A_VR x_R, with x_R
// the values the patch does not update (its dropped end nodes and the traces
// of the cells beyond them).  So no operator pass runs over the tile: with the
// 1-D relation (HostTables) S^T L v = Lambda S^T M v + gp v_c + gt u (v_c the
// dropped end values of a line, u the outer traces),
//   S3 x_V = Lambda^{-1} [S3^T b - sum_dir (gp (x) c_dir + gt (x) t_dir)] - w,
// where c_dir, t_dir are the dropped end layer and the outer trace of the two
// patch faces of direction dir, transformed by S^T M along the face, and w is
// S3^T M3 of the dropped nodes.  The forward passes S_z^T, S_y^T, S_x^T run over
// z-, y-, x-lines and each adds the faces of its own direction, where they are
// scalars of the lane: the masses alone act on a face along the directions
// whose S^T pass still follows.  On the way back w is taken off face by face
// (x-faces in the eigenbasis along y and z, y-faces in it along z, z-faces as
// plain nodal values), so that every dropped node counts once.
//
// What bounds it: the volume passes are six contractions of E-point lines
// instead of thirteen, five phases and one tile of LDS instead of seven and
// two; the faces cost O(E^2) lines per patch.

// Lines whose registers (E values, several lines live at once) leave no room for
// loads issued ahead: there the loads stay with their use.
template <typename T>
constexpr bool kGsTight = (D == 3) && E >= 10;

// Value of a patch face pair at one point: sum and difference of the left and
// right layer; an end that is not dropped counts as zero (type 0 uses both
// parts, types 1 and 2 the sum alone).
template <typename T>
struct FacePair {
  T s, d;
};
template <typename T>
__device__ __forceinline__ FacePair<T> face_sum(int ty, T l, T r) {
  return FacePair<T>{((ty & 1) ? T(0) : l) + ((ty & 2) ? T(0) : r), l - r};
}

// Outputs of a line that half H of a two-wave patch forms (H < 0: one wave, all):
// the even or the odd eigenvectors of an interior line forward, mirrored pairs of
// nodes back, as the even-odd forms share their sums; the same for every type.
template <int H>
__device__ __forceinline__ constexpr bool own_coef(int q) {
  return H < 0 || (q < kEOH) == (H == 0);
}
template <int H>
__device__ __forceinline__ constexpr bool own_pair(int k) {  // nodes 1 + k and E - 2 - k
  return H < 0 || (k < (kEOH + 1) / 2) == (H == 0);
}
template <int H>
__device__ __forceinline__ constexpr bool own_node(int p) {
  return H < 0 || (p == 0 || p == E - 1 ? H == 1 : own_pair<H>(p <= kEOH ? p - 1 : E - 2 - p));
}
template <int H, typename T>
__device__ __forceinline__ void store_coefs(T* s, int base, int stride, const Line<T>& L) {
#pragma unroll
  for (int q = 0; q < E; ++q)
    if (own_coef<H>(q)) s[base + q * stride] = L.v[q];
}
template <int H, typename T>
__device__ __forceinline__ void store_nodes(T* s, int base, int stride, const Line<T>& L) {
#pragma unroll
  for (int p = 0; p < E; ++p)
    if (own_node<H>(p)) s[base + p * stride] = L.v[p];
}

// o = S^T v - gp F - gt U, the ends and traces of the line as face pairs
template <typename T, int TY, bool OPQ, int H>
__device__ __forceinline__ void line_fwd_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, const FacePair<T>& F,
                                           const FacePair<T>& U, Line<T>& o) {
  using B = FDB<SP_DIR, TY>;
  const Coef<T> S = pass_coef<T, OPQ>(t->S[TY]), gp = pass_coef<T, OPQ>(t->gp[TY]),
                gt = pass_coef<T, OPQ>(t->gt[TY]);
  T vp[kEOH], vm[kEOH];
  if constexpr (kEO && TY == 0) eo_split<T>(v, vp, vm);
#pragma unroll
  for (int q = 0; q < E; ++q) {
    if (!own_coef<H>(q)) continue;
    if (q >= B::QN) {
      o.v[q] = T(0);
      continue;
    }
    const bool odd = TY == 0 && q >= kEOH;
    T s = -gp[q] * (odd ? F.d : F.s);
    s -= gt[q] * (odd ? U.d : U.s);
    if constexpr (kEO && TY == 0) {
#pragma unroll
      for (int k = 0; k < kEOH; ++k) s += S[(1 + k) * E + q] * (odd ? vm[k] : vp[k]);
    } else {
#pragma unroll
      for (int p = B::PLO; p < B::PHI; ++p) s += S[p * E + q] * v.v[p];
    }
    o.v[q] = s;
  }
}
// o = S (v - gm W), W the dropped end nodes of the line
template <typename T, int TY, bool OPQ, int H>
__device__ __forceinline__ void line_back_t(const Tab<K, T>* __restrict__ t, Line<T>& v, const FacePair<T>& W,
                                            Line<T>& o) {
  using B = FDB<SP_DIR, TY>;
  const Coef<T> gm = pass_coef<T, OPQ>(t->gm[TY]);
#pragma unroll
  for (int q = 0; q < B::QN; ++q) v.v[q] -= gm[q] * ((TY == 0 && q >= kEOH) ? W.d : W.s);
  const Coef<T> S = pass_coef<T, OPQ>(t->S[TY]);
  if constexpr (kEO && TY == 0) {
    // written in node order, as the other types write theirs: the compiler
    // then merges the branches' stores into one line without a
    // runtime-indexed copy of it (which would live in scratch)
    T e[kEOH], d[kEOH];
#pragma unroll
    for (int k = 0; k < kEOH; ++k) {
      if (!own_pair<H>(k)) continue;
      e[k] = d[k] = T(0);
#pragma unroll
      for (int q = 0; q < kEOH; ++q) e[k] += S[(1 + k) * E + q] * v.v[q];
#pragma unroll
      for (int q = 0; q < kEOH; ++q) d[k] += S[(1 + k) * E + kEOH + q] * v.v[kEOH + q];
    }
    if (own_node<H>(0)) o.v[0] = T(0);
#pragma unroll
    for (int k = 0; k < kEOH; ++k)
      if (own_pair<H>(k)) o.v[1 + k] = e[k] + d[k];
#pragma unroll
    for (int k = kEOH - 1; k >= 0; --k)
      if (own_pair<H>(k)) o.v[E - 2 - k] = e[k] - d[k];
    if (own_node<H>(E - 1)) o.v[E - 1] = T(0);
    return;
  }
#pragma unroll
  for (int p = 0; p < E; ++p) {
    if (!own_node<H>(p)) continue;
    T s = T(0);
    if (p >= B::PLO && p < B::PHI) {
#pragma unroll
      for (int q = 0; q < B::QN; ++q) s += S[p * E + q] * v.v[q];
    }
    o.v[p] = s;
  }
}
// the x-pass: forward, 1 / (sum lambda), the x-faces' part of w, back; sums: the
// inverse eigenvalue sums of the line, read into r where they were not before
template <typename T, int TY, bool OPQ, typename Sums>
__device__ __forceinline__ void line_turn_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, const FacePair<T>& F,
                                            const FacePair<T>& U, const FacePair<T>& W, T inv_scale,
                                            const T (&r)[E], Sums sums, Line<T>& o) {
  Line<T> w;
  line_fwd_t<T, TY, OPQ, -1>(t, v, F, U, w);
  sums();
#pragma unroll
  for (int q = 0; q < FDB<SP_DIR, TY>::QN; ++q) w.v[q] = w.v[q] * (inv_scale * r[q]);
  line_back_t<T, TY, OPQ, -1>(t, w, W, o);
}
// o = S^T M v over the whole line
template <typename T, int TY, int H>
__device__ __forceinline__ void line_MS_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, Line<T>& o) {
  const Coef<T> S = pass_coef<T, true>(t->MS[TY]);
  T vp[n], vm[n];
  if constexpr (TY == 0) {  // even and odd eigenvectors: half columns on sums and differences
#pragma unroll
    for (int p = 0; p < n; ++p) {
      vp[p] = v.v[p] + v.v[E - 1 - p];
      vm[p] = v.v[p] - v.v[E - 1 - p];
    }
  }
#pragma unroll
  for (int q = 0; q < E; ++q) {
    if (!own_coef<H>(q)) continue;
    T s = T(0);
    if (q < FDB<SP_DIR, TY>::QN) {
      if constexpr (TY == 0) {
#pragma unroll
        for (int p = 0; p < n; ++p) s += S[p * E + q] * (q < kEOH ? vp[p] : vm[p]);
      } else {
#pragma unroll
        for (int p = 0; p < E; ++p) s += S[p * E + q] * v.v[p];
      }
    }
    o.v[q] = s;
  }
}

// The passes for a patch type known at compile time (INT: an interior patch,
// type 0 in every direction) or not.  Type 3, both ends on the boundary, does
// not occur: the smoothers run on meshes of at least four cells a direction.
template <typename T, bool INT, int H>
struct GsLine {
  // an interior patch's passes share S and the couplings where these fit in
  // the scalar registers
  static constexpr bool OPQ = !INT || (2 * kEOH * ((kEO ? kEOH : 2 * kEOH) + 3)) * (int)sizeof(T) > 4 * 72;
  static __device__ __forceinline__ void fwd(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v,
                                             const FacePair<T>& F, const FacePair<T>& U, Line<T>& o) {
    if constexpr (INT) return line_fwd_t<T, 0, OPQ, H>(t, v, F, U, o);
    switch (ty) {
      case 0: line_fwd_t<T, 0, OPQ, H>(t, v, F, U, o); break;
      case 1: line_fwd_t<T, 1, OPQ, H>(t, v, F, U, o); break;
      default: line_fwd_t<T, 2, OPQ, H>(t, v, F, U, o); break;
    }
  }
  static __device__ __forceinline__ void back(const Tab<K, T>* __restrict__ t, int ty, Line<T>& v,
                                              const FacePair<T>& W, Line<T>& o) {
    if constexpr (INT) return line_back_t<T, 0, OPQ, H>(t, v, W, o);
    switch (ty) {
      case 0: line_back_t<T, 0, OPQ, H>(t, v, W, o); break;
      case 1: line_back_t<T, 1, OPQ, H>(t, v, W, o); break;
      default: line_back_t<T, 2, OPQ, H>(t, v, W, o); break;
    }
  }
  template <typename Sums>
  static __device__ __forceinline__ void turn(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v,
                                              const FacePair<T>& F, const FacePair<T>& U, const FacePair<T>& W,
                                              T inv_scale, const T (&r)[E], Sums sums, Line<T>& o) {
    if constexpr (INT) return line_turn_t<T, 0, OPQ>(t, v, F, U, W, inv_scale, r, sums, o);
    switch (ty) {
      case 0: line_turn_t<T, 0, OPQ>(t, v, F, U, W, inv_scale, r, sums, o); break;
      case 1: line_turn_t<T, 1, OPQ>(t, v, F, U, W, inv_scale, r, sums, o); break;
      default: line_turn_t<T, 2, OPQ>(t, v, F, U, W, inv_scale, r, sums, o); break;
    }
  }
  static __device__ __forceinline__ void ms(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v, Line<T>& o) {
    if constexpr (INT) return line_MS_t<T, 0, H>(t, v, o);
    switch (ty) {
      case 0: line_MS_t<T, 0, H>(t, v, o); break;
      case 1: line_MS_t<T, 1, H>(t, v, o); break;
      default: line_MS_t<T, 2, H>(t, v, o); break;
    }
  }
};

// The scalar cache starts every launch empty, and a pass that reads its
// coefficients where it needs them waits for the L2 each time.  warm_coef reads
// one word of every cache line of [p, p + count) at the start, together with
// the first vector loads; the caller hands the combined words to warm_wait,
// behind those loads.
template <typename T>
__device__ __forceinline__ unsigned warm_coef(const T* p, int count) {
  const Coef<unsigned> w = (Coef<unsigned>)(unsigned long long)p;
  unsigned x = 0;
#pragma unroll
  for (int i = 0; i < count * (int)sizeof(T) / 4; i += 16) x ^= w[i];
  return x;
}
__device__ __forceinline__ void warm_wait(unsigned x) { asm volatile("" ::"s"(x)); }

// i / DIV for the small non-negative indices of a patch (24-bit multiply and
// shift; exact below 512 for the divisors 2..64)
template <int DIV>
__device__ __forceinline__ int small_div(int i) {
  static_assert(DIV >= 2 && DIV <= 64, "checked divisors");
  if constexpr ((DIV & (DIV - 1)) == 0) return (unsigned)i / DIV;
  return (int)(__umul24((unsigned)i, 65536u / DIV + 1) >> 16);
}

// Element o of a vector part that starts at the (wave-uniform) address p:
// 32-bit offsets, so that the loads take the scalar base and one lane offset.
// The offsets span at most three planes of cells (3 N^(D-1) (k+1)^D entries),
// below 4 GB for every vector that fits the device.
template <typename T>
__device__ __forceinline__ const T& at32(const T* p, unsigned o) {
  return *(const T*)((const char*)p + (size_t)(o * (unsigned)sizeof(T)));
}
template <typename T>
__device__ __forceinline__ T& at32(T* p, unsigned o) {
  return *(T*)((char*)p + (size_t)(o * (unsigned)sizeof(T)));
}

// One patch of one colour (see smooth_body for the arguments).  MODE 2 (the
// paper's residual) differs only in the outer trace, for which it takes the
// patch's own end value.  ZERO: x = 0 on entry, so there are no faces, and
// every node of the tile is written.  INT: the patch is an interior one.
// GUARD: the launch has patches that look at their old values, this one if guard.
// H: half of a two-wave patch (k_smooth_split), -1: the patch is one wave's work.
//
// Order of the loads: the face layers and lines, then (where the registers
// allow it) b, all before the first of them is used -- one memory round trip.
template <typename T, int MODE, bool ZERO, bool INT, bool GUARD, int H = -1>
__device__ __forceinline__ void gs_body(const Tab<K, T>* __restrict__ t, int N, const PatchPos& P, T scale,
                                        T inv_scale, T* __restrict__ xr, const T* __restrict__ br, bool active,
                                        int lane, T* A, bool guard) {
  static_assert(NL == TPP && NF == TPP, "one line and one face node per lane");
  static_assert(H < 0 || (D == 3 && TPP % 64 == 0), "halves of whole waves");
  using L1 = GsLine<T, INT, H>;
  const int tyx = INT ? 0 : P.ty[0], tyy = INT ? 0 : P.ty[1], tyl = INT ? 0 : P.ty[D - 1];
  // The lane's coordinates (a, q): in 3-D the lanes run through the plane cell
  // by cell (cell and node an, am of a; qn, qm of q), as the vectors do, so that
  // the loads and stores of a plane touch the fewest cache lines: the cache
  // accesses of the row-by-row order (1030 a wave for 3-D Q4 in FP32) were
  // what bound the launch there.
  int an, am, qn = 0, qm = 0;
  if constexpr (D == 3) {
    const int cell = small_div<n * n>(lane), in = lane - cell * (n * n);
    qm = small_div<n>(in);
    am = in - qm * n;
    an = cell & 1;
    qn = cell >> 1;
  } else {
    an = small_div<n>(lane);
    am = lane - an * n;
  }
  const int a = an * n + am, q = qn * n + qm;
  // the lane's line along the last direction: node p of cell c at
  // x0 + c lc + lo + (p % n) ln
  constexpr int ln = (D == 3) ? n * n : n;
  const unsigned cy = (unsigned)N * NC;                       // next cell in y
  const unsigned lc = (D == 3) ? (unsigned)N * cy : cy;       // next cell in the last direction
  const long long p0 = cell_index(N, P.lo[0], P.lo[1], D == 3 ? P.lo[2] : 0) * NC;
  T* x0 = xr + p0;
  T* x1 = x0 + lc;
  const T *b0 = br + p0, *b1 = b0 + lc;
  const unsigned lo = (unsigned)(an * NC + am) + (D == 3 ? (unsigned)qn * cy + (unsigned)(n * qm) : 0u);
  Line<T> bl;
  auto load_b = [&]() {
#pragma unroll
    for (int p = 0; p < E; ++p) bl.v[p] = at32(p < n ? b0 : b1, lo + (p % n) * ln);
  };
  // The new values do not depend on the old ones on V, yet a NaN or an infinity
  // among these must not vanish: nonf, 0 or NaN, joins the lane's load line, and the
  // contractions carry it over the patch, as those of a residual do.
  T nonf = T(0);
  // faces of the last direction (Fl, Ul; Wl nodal) and of the x-direction (F is
  // scale W), and in 3-D of the y-direction (Wy in the eigenbasis along z)
  FacePair<T> Fl{}, Ul{}, Wl{}, Ux{}, Wx{}, Fy{}, Uy{}, Wy{};
  constexpr bool TIGHT = kGsTight<T>;
  // mass rows of the lane's nodes in x and (3-D) y: short ones by the first
  // loads, long ones (registers, cache accesses) from LDS at their use
  constexpr bool ROWLDS = D == 3 && n > 4;
  // (where the types are known to be uniform and the tables short; an interior
  // patch reads too little for it to show)
  constexpr bool WARM = !INT && TPP % 64 == 0 && E * E * (int)sizeof(T) <= 512;
  unsigned warm = 0;
  if constexpr (WARM) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int ty = i == 0 ? tyx : i == 1 ? tyy : tyl;
      warm ^= warm_coef<T>(t->S[ty], E * E) ^ warm_coef<T>(t->gp[ty], E) ^ warm_coef<T>(t->gt[ty], E) ^
              warm_coef<T>(t->gm[ty], E);
      if (!ZERO && D == 3 && i > 0) warm ^= warm_coef<T>(t->MS[ty], E * E);
    }
  }
  if constexpr (!ZERO) {
    T rowx[n], rowy[n];
    if constexpr (!ROWLDS) mass_row<T>(am, rowx);
    if constexpr (!ROWLDS && D == 3) mass_row<T>(qm, rowy);
    // raw layers of the last direction at this lane's node: left end, left
    // trace, right end, right trace (a side on the domain boundary reads the
    // patch's own node; its value is not used)
    const bool ownl = MODE == 2 || (tyl & 1), ownr = MODE == 2 || (tyl & 2);
    T raw[4] = {T(0), T(0), T(0), T(0)};
    Line<T> old{};
    if (GUARD && active && guard) {
#pragma unroll
      for (int p = 0; p < E; ++p) old.v[p] = at32(p < n ? x0 : x1, lo + (p % n) * ln);
    }
    if (active) {
      raw[0] = at32(x0, lo);
      if (H <= 0) raw[1] = ownl ? raw[0] : at32(x0 - lc, lo + K * ln);
      raw[2] = at32(x1, lo + K * ln);
      if (H != 0) raw[3] = ownr ? raw[2] : at32(x1 + lc, lo);
    }
    if constexpr (D == 3) {
      // lines along z of the y-faces (field f = 0..3: left end, left trace,
      // right end, right trace; i = px) and x-faces (f = 4..7; i = py):
      // S_z^T M_z into planes f; the raw z-layers into planes 8..11
      if (active) {
        const T* xm = x0 - cy - NC;
        if (ROWLDS && H <= 0 && lane < n * n) A[kGsM + lane] = kMassRows<T>.v[lane];
        // (3-D Q2 has more lines than lanes: all of its loads go first)
        constexpr int NIT = (8 * E + TPP - 1) / TPP;
        Line<T> v[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int li = it * TPP + lane;
          if (8 * E % TPP != 0 && li >= 8 * E) break;
          const int f = small_div<E>(li), i = li - f * E;
          const int in = small_div<n>(i), im = i - in * n;
          const bool xdir = f >= 4, right = (f & 2) != 0;
          const bool trace = (f & 1) && MODE != 2 && !((xdir ? tyx : tyy) & (right ? 2 : 1));
          // the layer's cell along the face normal (lo is 1: xm lies one cell
          // below) and its node there; i runs over the tangential direction
          const unsigned cn = (right ? 2u : 1u) + (trace ? (right ? 1u : ~0u) : 0u);
          const unsigned kn = (right != trace) ? K : 0;
          const unsigned o = xdir ? cn * NC + kn + (unsigned)(in + 1) * cy + n * im
                                  : cn * cy + n * kn + (unsigned)((in + 1) * NC + im);
#pragma unroll
          for (int p = 0; p < E; ++p) v[it].v[p] = at32(p < n ? xm : xm + lc, o + (p % n) * ln);
        }
        if constexpr (!TIGHT) load_b();
        if constexpr (WARM) warm_wait(warm);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int li = it * TPP + lane;
          if (8 * E % TPP != 0 && li >= 8 * E) break;
          const int f = small_div<E>(li), i = li - f * E;
          Line<T> w;
          L1::ms(t, tyl, v[it], w);
          store_coefs<H>(A, f * SZ + i, SY, w);
        }
#pragma unroll
        for (int f = 0; f < 4; ++f)
          if (H < 0 || f / 2 == H) A[(8 + f) * SZ + q * SY + a] = raw[f];
        if (GUARD && guard) {
#pragma unroll
          for (int p = 0; p < E; ++p) nonf += T(0) * old.v[p];
        }
      }
      __syncthreads();
      // M_x on the z-layers (planes 8..11 -> 12..15) and on the y-faces (this
      // lane: px = a, z-coefficient q), S_y^T M_y on the x-faces' lines
      if (active) {
        const T* rx = A + q * SY + an * n;
        T ym[4];
        if constexpr (ROWLDS) {
#pragma unroll
          for (int nu = 0; nu < n; ++nu) rowx[nu] = A[kGsM + am * n + nu];
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          T s = T(0), u = T(0);
#pragma unroll
          for (int nu = 0; nu < n; ++nu) s += rowx[nu] * rx[(8 + f) * SZ + nu];
#pragma unroll
          for (int nu = 0; nu < n; ++nu) u += rowx[nu] * rx[f * SZ + nu];
          if (H <= 0) A[(12 + f) * SZ + q * SY + a] = s;
          ym[f] = scale * u;
          if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
        }
        Fy = face_sum<T>(tyy, ym[0], ym[2]);
        Uy = face_sum<T>(tyy, ym[1], ym[3]);
        Wy = face_sum<T>(tyy, A[0 * SZ + q * SY + a], A[2 * SZ + q * SY + a]);
        // x-faces: one line per lane, on the last 4 E lanes
        constexpr int first = TPP > 4 * E ? TPP - 4 * E : 0;
#pragma unroll
        for (int li0 = 0; li0 < 4 * E; li0 += TPP) {
          const int li = li0 + lane - first;
          if (H == 0 || li < 0 || li >= 4 * E) continue;
          const int f = small_div<E>(li);
          T* r = A + (4 + f) * SZ + (li - f * E) * SY;
          Line<T> v, w;
          load_line(r, 0, 1, v);
          GsLine<T, INT, -1>::ms(t, tyy, v, w);  // whole lines, in place
          store_line(r, 0, 1, w);
        }
        if constexpr (TIGHT) load_b();
      }
      __syncthreads();
      // M_y on the z-layers; the x-faces of this lane's x-line (qy, qz) = (a, q)
      if (active) {
        const T* ry = A + qn * n * SY + a;
        T zm[4], xm[4];
        if constexpr (ROWLDS) {
#pragma unroll
          for (int nu = 0; nu < n; ++nu) rowy[nu] = A[kGsM + qm * n + nu];
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          T s = T(0);
#pragma unroll
          for (int nu = 0; nu < n; ++nu) s += rowy[nu] * ry[(12 + f) * SZ + nu * SY];
          zm[f] = scale * s;
          xm[f] = A[(4 + f) * SZ + q * SY + a];
          if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
        }
        Fl = face_sum<T>(tyl, zm[0], zm[2]);
        Ul = face_sum<T>(tyl, zm[1], zm[3]);
        Wx = face_sum<T>(tyx, xm[0], xm[2]);
        Ux = face_sum<T>(tyx, scale * xm[1], scale * xm[3]);
      }
    } else {
      // x-layers at py = lane, transformed by S_y^T M_y below
      const bool xl = MODE == 2 || (tyx & 1), xrt = MODE == 2 || (tyx & 2);
      T col[E];
      if (active) {
#pragma unroll
        for (int p = 0; p < E; ++p) col[p] = at32(t->MS[tyl], (unsigned)(p * E + a));
        const unsigned lx = (unsigned)an * cy + (unsigned)(n * am);
        const T* xm = x0 - NC;
        const T u0 = at32(xm, lx + NC), u2 = at32(xm, lx + 2 * NC + K);
        const T u1 = xl ? u0 : at32(xm, lx + K), u3 = xrt ? u2 : at32(xm, lx + 3 * NC);
        load_b();
        if constexpr (WARM) warm_wait(warm);
        A[4 * E + a] = u0;
        A[5 * E + a] = u1;
        A[6 * E + a] = u2;
        A[7 * E + a] = u3;
#pragma unroll
        for (int f = 0; f < 4; ++f) A[f * E + a] = raw[f];
        if (GUARD && guard) {
#pragma unroll
          for (int p = 0; p < E; ++p) nonf += T(0) * old.v[p];
        }
      }
      __syncthreads();
      if (active) {
        T ym[4], xm[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          T s = T(0);
#pragma unroll
          for (int nu = 0; nu < n; ++nu) s += rowx[nu] * A[f * E + an * n + nu];
          ym[f] = scale * s;
        }
        // col: this lane's eigenvector qy = a, its column of S^T M
#pragma unroll
        for (int p = 0; p < E; ++p) {
#pragma unroll
          for (int f = 0; f < 4; ++f) xm[f] += col[p] * A[(4 + f) * E + p];
        }
        Fl = face_sum<T>(tyl, ym[0], ym[2]);
        Ul = face_sum<T>(tyl, ym[1], ym[3]);
        Wx = face_sum<T>(tyx, xm[0], xm[2]);
        Ux = face_sum<T>(tyx, scale * xm[1], scale * xm[3]);
      }
    }
    Wl = face_sum<T>(tyl, raw[0], raw[2]);
    __syncthreads();  // the tile takes the place of the face fields
  } else {
    if (active) load_b();
    if constexpr (WARM) warm_wait(warm);
  }
  // where this lane's lines along x, y and the last direction start in the tile
  const int bx = a * SY + q * SZ, by = a + q * SZ, bz = (D == 3) ? a + q * SY : a;
  constexpr int sl = (D == 3) ? SZ : SY;
  // two waves read whole lines and each writes its outputs: two tiles in turn
  T* Z = A;
  T* B = H < 0 ? Z : A + TS;
  // inverse eigenvalue sums of the lane's x-line (qy, qz) = (a, q): asked for two
  // passes ahead (3-D Q2 FP64, 8^3 cells: a step 45.2 -> 43.7 us), or where registers
  // are short only when needed
  constexpr bool LATE = TIGHT && H < 0;
  T r[E];
  auto load_sums = [&]() {
    const T* rs = &at32(t->rs[0][(D == 3) ? (tyx * 4 + tyy) * 4 + tyl : tyx * 4 + tyy], (unsigned)lane);
#pragma unroll
    for (int c = 0; c < E; ++c)
      if (own_coef<H>(c)) r[c] = rs[c * NL];
  };
  auto late_sums = [&]() {
    if constexpr (LATE) {
      __builtin_amdgcn_sched_barrier(0);
      load_sums();
    }
  };
  // last direction: S^T b - its faces
  if (active) {
    Line<T> o;
    if constexpr (!LATE) load_sums();
    if constexpr (GUARD) bl.v[n] += nonf;  // node n is in every V
    L1::fwd(t, tyl, bl, Fl, Ul, o);
    store_coefs<H>(Z, bz, sl, o);
  }
  __syncthreads();
  if constexpr (D == 3) {
    if (active) {
      Line<T> v, o;
      load_line(Z, by, SY, v);
      L1::fwd(t, tyy, v, Fy, Uy, o);
      store_coefs<H>(B, by, SY, o);
    }
    __syncthreads();
  }
  if (active) {
    const FacePair<T> Fx{scale * Wx.s, scale * Wx.d};
    Line<T> v, o;
    load_line(B, bx, 1, v);
    if constexpr (H < 0) {
      L1::turn(t, tyx, v, Fx, Ux, Wx, inv_scale, r, late_sums, o);
    } else {
      L1::fwd(t, tyx, v, Fx, Ux, o);
#pragma unroll
      for (int c = 0; c < E; ++c)
        if (own_coef<H>(c)) o.v[c] = o.v[c] * (inv_scale * r[c]);
    }
    store_coefs<H>(Z, bx, 1, o);
  }
  __syncthreads();
  if constexpr (H >= 0) {
    if (active) {
      Line<T> v, o;
      load_line(Z, bx, 1, v);
      L1::back(t, tyx, v, Wx, o);
      store_nodes<H>(B, bx, 1, o);
    }
    __syncthreads();
  }
  if constexpr (D == 3) {
    if (active) {
      Line<T> v, o;
      load_line(B, by, SY, v);
      L1::back(t, tyy, v, Wy, o);
      store_nodes<H>(Z, by, SY, o);
    }
    __syncthreads();
  }
  // last direction back; only the nodes of V are written (ZERO: all of them,
  // the others as the zeros they hold)
  const bool keep_line = ZERO || ((a > 0 || (tyx & 1)) && (a < E - 1 || (tyx & 2)) &&
                                  (D == 2 || ((q > 0 || (tyy & 1)) && (q < E - 1 || (tyy & 2)))));
  if (active && keep_line) {
    Line<T> v, o;
    load_line(Z, bz, sl, v);
    L1::back(t, tyl, v, Wl, o);
#pragma unroll
    for (int p = 0; p < E; ++p) {
      if (!own_node<H>(p) || (!ZERO && ((p == 0 && !(tyl & 1)) || (p == E - 1 && !(tyl & 2))))) continue;
      at32(p < n ? x0 : x1, lo + (p % n) * ln) = o.v[p];
    }
  }
}

// One patch (pid of grid g, right-hand side rhs) of one colour; lane = thread
// within the patch, sm = the patch's LDS.  Every thread of the workgroup calls
// this (barriers inside), with pid >= g.npatch for idle slots.
// UNI: no wave holds lanes of patches of different types (the barriers of the
// two paths it then may take are the same in number).
template <typename T, int MODE, bool PREFETCH, bool ZERO, bool UNI = (TPP % 64 == 0), bool GUARD = false>
__device__ __forceinline__ void smooth_body(const Tab<K, T>* __restrict__ t, const PatchGrid& g, T scale,
                                            T inv_scale, const T* __restrict__ xin, T* __restrict__ xout,
                                            const T* __restrict__ b, long long ndof, int pid, int lane,
                                            T* sm, int rhs) {
  if constexpr (kDirect<MODE>) {
    const bool act = pid < g.npatch;
    // an idle slot of a right-hand-side-packed workgroup takes the position of
    // the others: slots that share a wave have to take one path
    const PatchPos Q = patch_pos(g, act ? pid : pid - g.npatch);
    T* xv = xout + (long long)rhs * ndof;
    const T* bv = b + (long long)rhs * ndof;
    if (UNI && (Q.ty[0] | Q.ty[1] | Q.ty[2]) == 0)
      gs_body<T, MODE, ZERO, true, GUARD>(t, g.N, Q, scale, inv_scale, xv, bv, act, lane, sm, g.guard == 2);
    else
      gs_body<T, MODE, ZERO, false, GUARD>(t, g.N, Q, scale, inv_scale, xv, bv, act, lane, sm, true);
  } else {
  constexpr bool FULL = (MODE == 3);
  constexpr int SP = FULL ? SP_FULL : (MODE == 4) ? SP_CLAMPED : SP_DIR;
  // operator-pass mode (side data)
  constexpr int OPM = FULL ? 0 : (MODE == 4) ? 2 : MODE > 4 ? MODE - 4 : MODE;
  const bool inrange = pid < g.npatch;
  T* A = sm;
  T* B = A + TS;
  T* ext = B + TS;
  const long long roff = (long long)rhs * ndof;
  T* xw = xout + roff;
  const T* xr = (FULL ? xin : xout) + roff;
  const T* br = b + roff;
  const PatchPos P = patch_pos(g, inrange ? pid : 0);
  bool whole = true;  // partial patches exist only in the Full kernel's launches
  if (FULL) {
#pragma unroll
    for (int i = 0; i < D; ++i) whole = whole && P.lo[i] >= 0 && P.lo[i] + 1 < g.N;
  }
  const bool active = inrange && whole;
  if (FULL && inrange && !whole) {
    // partial patch: copy the rows of its in-domain cells
    for (int i = lane; i < NL; i += TPP) {
      const int py = i % E, pz = i / E;
      const int cy = P.lo[1] + py / n;
      const int cz = (D == 3) ? P.lo[2] + pz / n : 0;
      if (cy < 0 || cy >= g.N || cz < 0 || cz >= g.N) continue;
      if (D == 2 && pz > 0) continue;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int cx = P.lo[0] + c;
        if (cx < 0 || cx >= g.N) continue;
        const long long row = cell_index(g.N, cx, cy, cz) * NC + (py % n) * n + ((D == 3) ? (pz % n) * n * n : 0);
#pragma unroll
        for (int a = 0; a < n; ++a) xw[row + a] = xr[row + a];
      }
    }
  }
  const int tyx = P.ty[0], tyy = P.ty[1], tyz = P.ty[2];
  // inverse eigenvalue sums of the lane's scaling line: read at the start in
  // 2-D (used by the first contraction phase), in 3-D only once the residual
  // is formed, so that they are not held through the operator passes (the
  // loads still overlap the X1 phase)
  T rsl[E];
  if (D == 2 && active) load_rs<T, SP>(t, P.ty, lane, rsl);
  Line<T> xl;  // the thread's x-line of x, kept for the final update
  // y-face couplings of the thread's y-line, read early from global (Dirichlet
  // kernels), and (PREFETCH) its line of b for the last operator pass: one
  // memory round trip less on the critical path of a patch, one tile more in
  // flight per patch
  if constexpr (ZERO) {
    // r = b, contracted with S^T along the last direction
#pragma unroll
    for (int p = 0; p < E; ++p) xl.v[p] = T(0);
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(D - 1, i, base, stride);
        Line<T> r, o;
        read_lastline<T>(br, g.N, P, i, r);
        line_St<T, SP>(t, (D == 3) ? tyz : tyy, r, o);
        store_line(A, base, stride, o);
      }
  } else {
    Line<T> bline;
    if (PREFETCH && active) read_lastline<T>(br, g.N, P, lane, bline);

    // residual r = b - A x on the last pass, contracted with S^T of that direction
    auto emit = [&](int l, int base, int stride, const Line<T>& v) {
      Line<T> r, o;
      if (PREFETCH) r = bline;
      else read_lastline<T>(br, g.N, P, l, r);
#pragma unroll
      for (int p = 0; p < E; ++p) r.v[p] -= scale * v.v[p];
      line_St<T, SP>(t, (D == 3) ? tyz : tyy, r, o);
      store_line(A, base, stride, o);
    };
    if constexpr (FULL && kFullOnApplyRF)
      apply_rf_body<T, RF_EMIT>(t, g, scale, xin, nullptr, nullptr, ndof, 0, pid, lane, A, rhs, active, xl, emit);
    else
      operator_passes<T, OPM, FULL && kFullRF>(t, xr, g.N, P, A, B, ext, lane, active, xl, emit);
  }
  __syncthreads();
  if constexpr (D == 3) {
    if (active) load_rs<T, SP>(t, P.ty, lane, rsl);
    // X1: S_x^T
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(0, i, base, stride);
        Line<T> v, o;
        load_line(A, base, stride, v);
        line_St<T, SP>(t, tyx, v, o);
        store_line(A, base, stride, o);
      }
    __syncthreads();
    // Y1: S_y^T, scale by 1/(sum lambda), S_y (one line per lane: TPP = NL)
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(1, i, base, stride);
        Line<T> v, o;
        load_line(A, base, stride, v);
        line_St<T, SP>(t, tyy, v, o);
#pragma unroll
        for (int q = 0; q < E; ++q) o.v[q] = o.v[q] * (inv_scale * rsl[q]);
        line_S<T, SP>(t, tyy, o, v);
        store_line(A, base, stride, v);
      }
    __syncthreads();
    // Z1: S_z
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(2, i, base, stride);
        Line<T> v, o;
        load_line(A, base, stride, v);
        line_S<T, SP>(t, tyz, v, o);
        store_line(A, base, stride, o);
      }
    __syncthreads();
  } else {
    // X1: S_x^T, scale, S_x (one line per lane: TPP = NL)
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(0, i, base, stride);
        Line<T> v, o;
        load_line(A, base, stride, v);
        line_St<T, SP>(t, tyx, v, o);
#pragma unroll
        for (int q = 0; q < E; ++q) o.v[q] = o.v[q] * (inv_scale * rsl[q]);
        line_S<T, SP>(t, tyx, o, v);
        store_line(A, base, stride, v);
      }
    __syncthreads();
    // Y1: S_y
    if (active)
      for (int i = lane; i < NL; i += TPP) {
        int base, stride;
        line_geom(1, i, base, stride);
        Line<T> v, o;
        load_line(A, base, stride, v);
        line_S<T, SP>(t, tyy, v, o);
        store_line(A, base, stride, o);
      }
    __syncthreads();
  }
  // X2 (3-D) / final x pass (2-D): x += S_x delta on the kept nodes, or, in
  // 3-D, x += delta with delta already in physical coordinates along x.
  if (active) {
    for (int i = lane; i < NL; i += TPP) {
      const int py = i % E, pz = i / E;
      const bool keep_line = FULL || ZERO ||
                             ((py > 0 || (tyy & 1)) && (py < E - 1 || (tyy & 2)) &&
                              (D == 2 || ((pz > 0 || (tyz & 1)) && (pz < E - 1 || (tyz & 2)))));
      if (!keep_line) continue;
      int base, stride;
      line_geom(0, i, base, stride);
      Line<T> dl;
      load_line(A, base, stride, dl);
      if constexpr (D == 3) {
        Line<T> o;
        line_S<T, SP>(t, tyx, dl, o);
        dl = o;
      }
      // whole rows: the dropped end nodes of a Dirichlet V_j are rewritten
      // with their unchanged value (delta is exactly zero there), so no
      // same-colour reader can observe a different value
      const long long row0 = xrow_offset(g.N, P, py, pz);
      Line<T> nx;
#pragma unroll
      for (int p = 0; p < E; ++p) nx.v[p] = xl.v[p] + dl.v[p];
      if (!FULL && !(tyx & 1)) nx.v[0] = xl.v[0];
      if (!FULL && !(tyx & 2)) nx.v[E - 1] = xl.v[E - 1];
#pragma unroll
      for (int a = 0; a < n; ++a) {
        xw[row0 + a] = nx.v[a];
        xw[row0 + NC + a] = nx.v[n + a];
      }
    }
  }
  }
}

// Waves per SIMD the register allocation of k_smooth aims at (1: no aim): for
// the direct form in 3-D the most an interior patch's passes allow without
// spilled vector registers (scalar ones spill to vector lanes: 95 for Q3 FP64, 121 for
// Q7 FP32).
template <typename T, int MODE, int THREADS, bool GUARD>
constexpr int smooth_waves() {
  if (D != 3 || !kDirect<MODE> || THREADS > 256) return 1;
  if (sizeof(T) == 8) return K <= 4 ? 4 : 2;
  return K <= 3 ? (GUARD ? 7 : 8) : K == 4 ? 6 : K == 6 ? 4 : 5;
}
// LDS a workgroup of several right-hand sides may take: half a CU's
constexpr int kPackedLDS = 80 * 1024;
template <typename T, int PPB, int MODE, bool PREFETCH, bool ZERO = false, bool RP = false, bool GUARD = false>
__global__ void __launch_bounds__(TPP * PPB, (smooth_waves<T, MODE, TPP * PPB, GUARD>()))
k_smooth(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, T inv_scale,
         const T* __restrict__ xin, T* __restrict__ xout, const T* __restrict__ b, long long ndof) {
  constexpr int PP = smooth_pp<MODE, T>();
  static_assert(!RP || PPB * PP * (int)sizeof(T) <= kPackedLDS, "right-hand sides packed for this variant's footprint");
  __shared__ T smem[PPB * PP];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  int pid, rhs;
  slot_work<PPB, RP>(g, slot, pid, rhs);
  // one patch per workgroup, or one patch for all its slots
  constexpr bool UNI = PPB == 1 || RP || TPP % 64 == 0;
  smooth_body<T, MODE, PREFETCH, ZERO, UNI, GUARD>(t, g, scale, inv_scale, xin, xout, b, ndof, pid, lane,
                                                   smem + slot * PP, rhs);
}


// ----------------------------------------------- split smoother (3-D)
// The clamped kernel's colour step with two waves per patch (TPP a multiple of
// 64): wave h of a patch owns, for every tile line, the outputs of cell h
// (indices h n .. h n + n - 1) -- or the eigen-coefficients q in that range in
// the fast-diagonalisation contractions -- while both waves read whole lines.
// The 1-D coefficients a wave needs stay wave-uniform, each output element is
// computed with the operations of the one-wave kernel in the same order (so
// the results are bitwise those of k_smooth), and a patch occupies twice the
// waves for the same LDS: more waves per SIMD to hide each other's latency.
// Phases that rewrite the tile they read put a barrier between the reads of
// both waves and the writes.
template <typename T>
struct Half {
  T v[n];
};

template <int H>
__device__ __forceinline__ constexpr bool half_end(int mu) { return H == 0 ? mu == 0 : mu == n - 1; }

// o = (blockdiag(M, M) v) on cell H; the patch-end output only if needEnd
template <typename T, int H>
__device__ __forceinline__ void half_mass(const Line<T>& v, Half<T>& o, bool needEnd) {
  if constexpr (kEOC) {
    T bl[n];
    cell_eo<T, true>(v, H, bl);
#pragma unroll
    for (int mu = 0; mu < n; ++mu) {
      if (half_end<H>(mu) && !needEnd) continue;
      o.v[mu] = bl[mu];
    }
    return;
  }
#pragma unroll
  for (int mu = 0; mu < n; ++mu) {
    if (half_end<H>(mu) && !needEnd) continue;
    T s = T(0);
#pragma unroll
    for (int nu = 0; nu < n; ++nu) s += T(kRef.M[mu * n + nu]) * v.v[H * n + nu];
    o.v[mu] = s;
  }
}

// o (+)= 1-D SIPG of the patch line v on cell H (the rows of line_sipg, in
// its order of operations)
template <typename T, int H, bool ACC>
__device__ __forceinline__ void half_sipg(const Tab<K, T>* __restrict__ t, const Line<T>& v,
                                          const Sides<T>& sd, Half<T>& o, bool needEnd) {
  if constexpr (kDiff<T>) {
    cell_sipg_diff<T, H, ACC>(t->sigma, v, sd, o.v, needEnd, needEnd);
    return;
  }
  const T sg = t->sigma;
  const T half = T(0.5);
  T bl[n];
  if constexpr (kEOC) cell_eo<T, false>(v, H, bl);
#pragma unroll
  for (int mu = 0; mu < n; ++mu) {
    if (half_end<H>(mu) && !needEnd) continue;
    T s = ACC ? o.v[mu] : T(0);
    if constexpr (kEOC) {
      s += bl[mu];
    } else {
#pragma unroll
      for (int nu = 0; nu < n; ++nu) s += T(kRef.Lcons[mu * n + nu]) * v.v[H * n + nu];
    }
    if (mu == 0) s += sg * v.v[H * n];
    if (mu == n - 1) s += sg * v.v[H * n + n - 1];
    o.v[mu] = s;
  }
  if constexpr (H == 0) {
    const T tR = v.v[n];
    T gR = T(0);
#pragma unroll
    for (int j = 0; j < n; ++j) gR += T(kRef.d0[j]) * v.v[n + j];
    T aL = sd.aL, bL = sd.bL;
    if (sd.bl) {
      T g0 = T(0);
#pragma unroll
      for (int j = 0; j < n; ++j) g0 += T(kRef.d0[j]) * v.v[j];
      aL = half * g0;
      bL = half * v.v[0];
    }
    if (!sd.bl && sd.lit) bL = -half * v.v[0];
    const T bLc = half * tR;
    if (needEnd) {
      o.v[0] += aL;
      o.v[0] += T(kRef.d0[0]) * bL + T(kRef.d1[0]) * bLc;
    }
    o.v[n - 1] += -sg * tR - half * gR;
#pragma unroll
    for (int mu = 1; mu < n; ++mu) o.v[mu] += T(kRef.d0[mu]) * bL + T(kRef.d1[mu]) * bLc;
  } else {
    const T tL = v.v[n - 1];
    T gL = T(0);
#pragma unroll
    for (int j = 0; j < n; ++j) gL += T(kRef.d1[j]) * v.v[j];
    T aR = sd.aR, bR = sd.bR;
    if (sd.br) {
      T g1 = T(0);
#pragma unroll
      for (int j = 0; j < n; ++j) g1 += T(kRef.d1[j]) * v.v[n + j];
      aR = -half * g1;
      bR = -half * v.v[E - 1];
    }
    if (!sd.br && sd.lit) bR = half * v.v[E - 1];
    const T bRc = -half * tL;
    o.v[0] += half * gL - sg * tL;
    if (needEnd) {
      o.v[n - 1] += aR;
      o.v[n - 1] += T(kRef.d0[n - 1]) * bRc + T(kRef.d1[n - 1]) * bR;
    }
#pragma unroll
    for (int mu = 0; mu < n - 1; ++mu) o.v[mu] += T(kRef.d0[mu]) * bRc + T(kRef.d1[mu]) * bR;
  }
}

// o[j] = sum_p S[p][q] v[p], q = H n + j (coefficients of line_St_t)
template <typename T, int TY, int SP, int H>
__device__ __forceinline__ void half_St_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, Half<T>& o) {
  using B = FDB<SP, TY>;
  const Coef<T> S = pass_coef<T, kOpaqueFD<T, SP>>(fd_S<T, SP>(t, TY));
#pragma unroll
  for (int j = 0; j < n; ++j) {
    const int q = H * n + j;
    T s = T(0);
    if (q < B::QN) {
#pragma unroll
      for (int p = B::PLO; p < B::PHI; ++p) s += S[p * E + q] * v.v[p];
    }
    o.v[j] = s;
  }
}
// o[j] = sum_q S[p][q] v[q], p = H n + j
template <typename T, int TY, int SP, int H>
__device__ __forceinline__ void half_S_t(const Tab<K, T>* __restrict__ t, const Line<T>& v, Half<T>& o) {
  using B = FDB<SP, TY>;
  const Coef<T> S = pass_coef<T, kOpaqueFD<T, SP>>(fd_S<T, SP>(t, TY));
#pragma unroll
  for (int j = 0; j < n; ++j) {
    const int p = H * n + j;
    T s = T(0);
    if (p >= B::PLO && p < B::PHI) {
#pragma unroll
      for (int q = 0; q < B::QN; ++q) s += S[p * E + q] * v.v[q];
    }
    o.v[j] = s;
  }
}
template <typename T, int SP, int H>
__device__ __forceinline__ void half_St(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v, Half<T>& o) {
  switch (ty) {
    case 0: half_St_t<T, 0, SP, H>(t, v, o); break;
    case 1: half_St_t<T, 1, SP, H>(t, v, o); break;
    case 2: half_St_t<T, 2, SP, H>(t, v, o); break;
    default: half_St_t<T, 3, SP, H>(t, v, o); break;
  }
}
template <typename T, int SP, int H>
__device__ __forceinline__ void half_S(const Tab<K, T>* __restrict__ t, int ty, const Line<T>& v, Half<T>& o) {
  switch (ty) {
    case 0: half_S_t<T, 0, SP, H>(t, v, o); break;
    case 1: half_S_t<T, 1, SP, H>(t, v, o); break;
    case 2: half_S_t<T, 2, SP, H>(t, v, o); break;
    default: half_S_t<T, 3, SP, H>(t, v, o); break;
  }
}

template <typename T>
__device__ __forceinline__ void store_half(T* s, int base, int stride, int H, const Half<T>& o) {
#pragma unroll
  for (int j = 0; j < n; ++j) s[base + (H * n + j) * stride] = o.v[j];
}

// last-direction (z) line of b, the cells of half H only
template <typename T>
__device__ __forceinline__ void read_lasthalf(const T* __restrict__ b, int N, const PatchPos& P, int l, int H,
                                              Half<T>& v) {
  const long long base = node_offset(N, P, l % E, l / E, 0) + (long long)H * N * N * NC;
#pragma unroll
  for (int j = 0; j < n; ++j) v.v[j] = b[base + j * (n * n)];
}

constexpr bool kSplitOK = (D == 3) && (TPP % 64 == 0);

template <typename T, int MODE, bool PREFETCH, bool ZERO, int H>
__device__ __forceinline__ void smooth_split_body(const Tab<K, T>* __restrict__ t, const PatchGrid& g,
                                                  T scale, T inv_scale, T* __restrict__ x,
                                                  const T* __restrict__ b, long long ndof, int pid,
                                                  int lane, T* sm, int rhs) {
  static_assert(MODE == 4, "clamped kernel");
  constexpr int SP = SP_CLAMPED;
  const bool active = pid < g.npatch;
  T* A = sm;
  T* B = A + TS;
  const long long roff = (long long)rhs * ndof;
  T* xr = x + roff;
  const T* br = b + roff;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  const int tyx = P.ty[0], tyy = P.ty[1], tyz = P.ty[2];
  // ends of this half's cell that lie on the patch boundary are needed only
  // on the domain boundary (Dirichlet and clamped spaces)
  const bool endx = (tyx & (H == 0 ? 1 : 2)) != 0;
  const bool endy = (tyy & (H == 0 ? 1 : 2)) != 0;
  const bool endz = (tyz & (H == 0 ? 1 : 2)) != 0;
  Half<T> xh;  // this half of the thread's x-line of x
  Half<T> bh;  // this half of the thread's z-line of b
  T rsh[n];    // inverse eigenvalue sums of this half of the lane's scaling line
  if (PREFETCH && active) read_lasthalf<T>(br, g.N, P, lane, H, bh);
  if constexpr (ZERO) {
#pragma unroll
    for (int j = 0; j < n; ++j) xh.v[j] = T(0);
    if (active) {
      // r = b: this half to A, then S_z^T over whole lines into B
      if (!PREFETCH) read_lasthalf<T>(br, g.N, P, lane, H, bh);
      int base, stride;
      line_geom(2, lane, base, stride);
      store_half(A, base, stride, H, bh);
    }
    __syncthreads();
  } else {
    // the clamped residual reads the patch cells alone: no traces of the
    // neighbours, the sides only say where the domain boundary is
    const Sides<T> sd = bare_sides<T>(P.lo[0], g.N, true), ysd = bare_sides<T>(P.lo[1], g.N, true);
    Line<T> xl;
    const int py = lane % E, pz = lane / E;
    const long long row0 = xrow_offset(g.N, P, py, pz);
    if (active) {
      read_xline<T>(xr, row0, xl);
    }
    // X0: a = M_x x, b = L_x x on this half -> A, B
    if (active) {
#pragma unroll
      for (int j = 0; j < n; ++j) xh.v[j] = xl.v[H * n + j];
      int base, stride;
      line_geom(0, lane, base, stride);
      Half<T> a, bb;
      half_mass<T, H>(xl, a, endx);
      half_sipg<T, H, false>(t, xl, sd, bb, endx);
      store_half(A, base, stride, H, a);
      store_half(B, base, stride, H, bb);
    }
    __syncthreads();
    // Y: c = M_y b + L_y a -> B, d = M_y a -> A (after both waves have read)
    Half<T> c, d;
    int ybase = 0, ystride = 0;
    if (active) {
      line_geom(1, lane, ybase, ystride);
      Line<T> a, bl;
      load_line(A, ybase, ystride, a);
      load_line(B, ybase, ystride, bl);
      half_mass<T, H>(bl, c, endy);
      half_sipg<T, H, true>(t, a, ysd, c, endy);
      half_mass<T, H>(a, d, endy);
    }
    __syncthreads();
    if (active) {
      store_half(B, ybase, ystride, H, c);
      store_half(A, ybase, ystride, H, d);
    }
    __syncthreads();
    // Z: y = M_z c + L_z d, r = b - scale y on this half -> A, then S_z^T
    if (active) {
      int base, stride;
      line_geom(2, lane, base, stride);
      Line<T> cl, dl;
      load_line(B, base, stride, cl);
      load_line(A, base, stride, dl);
      const Sides<T> zsd = bare_sides<T>(P.lo[2], g.N, true);
      Half<T> y;
      half_mass<T, H>(cl, y, endz);
      half_sipg<T, H, true>(t, dl, zsd, y, endz);
      if (!PREFETCH) read_lasthalf<T>(br, g.N, P, lane, H, bh);
#pragma unroll
      for (int j = 0; j < n; ++j) bh.v[j] -= scale * y.v[j];
    }
    __syncthreads();
    if (active) {
      int base, stride;
      line_geom(2, lane, base, stride);
      store_half(A, base, stride, H, bh);
    }
    __syncthreads();
  }
  // (the eigenvalue sums are read only now, not held through the residual
  // passes; their loads overlap the next two phases)
  if (active) {
    T rsl[E];
    load_rs<T, SP>(t, P.ty, lane, rsl);
#pragma unroll
    for (int j = 0; j < n; ++j) rsh[j] = rsl[H * n + j];
  }
  // S_z^T over the whole residual line -> B
  if (active) {
    int base, stride;
    line_geom(2, lane, base, stride);
    Line<T> r;
    load_line(A, base, stride, r);
    Half<T> o;
    half_St<T, SP, H>(t, tyz, r, o);
    store_half(B, base, stride, H, o);
  }
  __syncthreads();
  // X1: S_x^T, B -> A
  if (active) {
    int base, stride;
    line_geom(0, lane, base, stride);
    Line<T> v;
    load_line(B, base, stride, v);
    Half<T> o;
    half_St<T, SP, H>(t, tyx, v, o);
    store_half(A, base, stride, H, o);
  }
  __syncthreads();
  // Y1a: S_y^T and 1/(sum lambda), A -> B
  if (active) {
    int base, stride;
    line_geom(1, lane, base, stride);
    Line<T> v;
    load_line(A, base, stride, v);
    Half<T> o;
    half_St<T, SP, H>(t, tyy, v, o);
#pragma unroll
    for (int j = 0; j < n; ++j) o.v[j] = o.v[j] * (inv_scale * rsh[j]);
    store_half(B, base, stride, H, o);
  }
  __syncthreads();
  // Y1b: S_y, B -> A
  if (active) {
    int base, stride;
    line_geom(1, lane, base, stride);
    Line<T> v;
    load_line(B, base, stride, v);
    Half<T> o;
    half_S<T, SP, H>(t, tyy, v, o);
    store_half(A, base, stride, H, o);
  }
  __syncthreads();
  // Z1: S_z, A -> B
  if (active) {
    int base, stride;
    line_geom(2, lane, base, stride);
    Line<T> v;
    load_line(A, base, stride, v);
    Half<T> o;
    half_S<T, SP, H>(t, tyz, v, o);
    store_half(B, base, stride, H, o);
  }
  __syncthreads();
  // X2: x += S_x delta on this half's cell row of the kept lines
  if (active) {
    const int py = lane % E, pz = lane / E;
    const bool keep_line = ZERO || ((py > 0 || (tyy & 1)) && (py < E - 1 || (tyy & 2)) &&
                                    (pz > 0 || (tyz & 1)) && (pz < E - 1 || (tyz & 2)));
    if (keep_line) {
      int base, stride;
      line_geom(0, lane, base, stride);
      Line<T> v;
      load_line(B, base, stride, v);
      Half<T> dl;
      half_S<T, SP, H>(t, tyx, v, dl);
      Half<T> nx;
#pragma unroll
      for (int j = 0; j < n; ++j) nx.v[j] = xh.v[j] + dl.v[j];
      if (H == 0 && !(tyx & 1)) nx.v[0] = xh.v[0];
      if (H == 1 && !(tyx & 2)) nx.v[n - 1] = xh.v[n - 1];
      const long long row = xrow_offset(g.N, P, py, pz) + (long long)H * NC;
#pragma unroll
      for (int j = 0; j < n; ++j) xr[row + j] = nx.v[j];
    }
  }
}

// Half H of a patch in any of the two-wave smoothers.  The direct form divides its
// lines' outputs over the halves by own_coef and own_node: what a wave does in a
// pass is halved, the x-pass becomes two, and a patch takes two tiles.  Bound by
// the latency of one patch's phases on levels of few patches, which is where the
// tuner takes it, V-cycles with two waves / one on every level: 3-D Q3 FP32 8^3 95.5 /
// 99.8 us, 16^3 183 / 190, FP64 116 / 120 and 219 / 223 us, Q7 FP32 8^3 365 / 401, 16^3 606 /
// 642 us; with many patches one wave is faster (Q3 FP64 32^3 475 / 434 us).  Both forms
// of an output have the operations of one wave in the same order, so the results
// are bitwise those of k_smooth.
template <typename T, int MODE, bool PREFETCH, bool ZERO, bool GUARD, int H>
__device__ __forceinline__ void smooth_half(const Tab<K, T>* __restrict__ t, const PatchGrid& g, T scale,
                                            T inv_scale, T* __restrict__ x, const T* __restrict__ b,
                                            long long ndof, int pid, int lane, T* sm, int rhs) {
  if constexpr (MODE == 4) {
    smooth_split_body<T, MODE, PREFETCH, ZERO, H>(t, g, scale, inv_scale, x, b, ndof, pid, lane, sm, rhs);
  } else {
    static_assert(kDirect<MODE>, "clamped kernel or direct form");
    const bool act = pid < g.npatch;
    const PatchPos P = patch_pos(g, act ? pid : 0);
    T* xv = x + (long long)rhs * ndof;
    const T* bv = b + (long long)rhs * ndof;
    if ((P.ty[0] | P.ty[1] | P.ty[2]) == 0)
      gs_body<T, MODE, ZERO, true, GUARD, H>(t, g.N, P, scale, inv_scale, xv, bv, act, lane, sm, g.guard == 2);
    else
      gs_body<T, MODE, ZERO, false, GUARD, H>(t, g.N, P, scale, inv_scale, xv, bv, act, lane, sm, true);
  }
}
// LDS per two-wave patch: two tiles
template <int MODE, typename T = double>
constexpr int split_pp() {
  return smooth_pp<MODE, T>() > 2 * TS ? smooth_pp<MODE, T>() : 2 * TS;
}

template <typename T, int PPB, int MODE, bool PREFETCH, bool ZERO = false, bool GUARD = false>
__global__ void __launch_bounds__(2 * TPP * PPB)
k_smooth_split(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, T inv_scale, T* __restrict__ x,
               const T* __restrict__ b, long long ndof) {
  constexpr int PP = split_pp<MODE, T>();
  __shared__ T smem[PPB * PP];
  const int w = (int)threadIdx.x / TPP;  // wave group: slot * 2 + half
  const int ws = kSplitOK ? __builtin_amdgcn_readfirstlane(w) : w;
  const int slot = ws / 2, h = ws % 2, lane = threadIdx.x % TPP;
  const int pid = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap) * PPB + slot;
  if (h == 0)
    smooth_half<T, MODE, PREFETCH, ZERO, GUARD, 0>(t, g, scale, inv_scale, x, b, ndof, pid, lane,
                                                   smem + slot * PP, blockIdx.y);
  else
    smooth_half<T, MODE, PREFETCH, ZERO, GUARD, 1>(t, g, scale, inv_scale, x, b, ndof, pid, lane,
                                                   smem + slot * PP, blockIdx.y);
}

// ------------------------------------------------- residual + restriction
// bc = P^T (b - A x): the colour-0 patch of level l is the set of children of
// one coarse cell, so its residual contracts with the stacked P^T per
// direction straight into that coarse cell.
// Q1, Q3 in 3-D: the operator pass takes the neighbour face data in registers
// (as the apply's shape 2): two tiles of LDS per patch, no face arrays.
constexpr bool kRestrictRF = (D == 3) && kZShfl;
constexpr int kRestrictPP = kRestrictRF ? 2 * TS : Smem<2, (D - 1) * 2 * 2 * NF>::per_patch;

template <typename T>
__device__ __forceinline__ void restrict_body(const Tab<K, T>* __restrict__ t, const PatchGrid& g, T scale,
                                              const T* __restrict__ x, const T* __restrict__ b,
                                              T* __restrict__ bc, long long ndof, long long ndof_c,
                                              int pid, int lane, T* sm, int rhs) {
  const bool active = pid < g.npatch;
  T* A = sm;
  T* B = A + TS;
  T* ext = B + TS;
  const long long roff = (long long)rhs * ndof;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  Line<T> xl;
  operator_passes<T, 0, kRestrictRF>(t, x + roff, g.N, P, A, B, ext, lane, active, xl,
                        [&](int l, int base, int stride, const Line<T>& v) {
                          Line<T> r;
                          read_lastline<T>(b + roff, g.N, P, l, r);
#pragma unroll
                          for (int nu = 0; nu < n; ++nu) {
                            T s = T(0);
#pragma unroll
                            for (int p = 0; p < E; ++p) s += T(kRef.P[p * n + nu]) * (r.v[p] - scale * v.v[p]);
                            A[base + nu * stride] = s;
                          }
                        });
  __syncthreads();
  restrict_tail<T>(g, P, A, bc, ndof_c, rhs, lane, active);
}

// The restriction after the last direction (its P^T values at the first n
// nodes of each last-direction line of A): P^T along y (3-D), then along x
// into the rows of the patch's coarse cell of bc.
template <typename T>
__device__ __forceinline__ void restrict_tail(const PatchGrid& g, const PatchPos& P, T* A, T* __restrict__ bc,
                                              long long ndof_c, int rhs, int lane, bool active) {
  if constexpr (D == 3) {
    // restrict along y: lines (px, pz < n)
    if (active)
      for (int i = lane; i < E * n; i += TPP) {
        const int px = i % E, pz = i / E;
        const int base = px + pz * SZ, stride = SY;
        Line<T> v;
        load_line(A, base, stride, v);
#pragma unroll
        for (int nu = 0; nu < n; ++nu) {
          T s = T(0);
#pragma unroll
          for (int p = 0; p < E; ++p) s += T(kRef.P[p * n + nu]) * v.v[p];
          A[base + nu * stride] = s;
        }
      }
    __syncthreads();
  }
  // restrict along x: lines (py < n, pz < n) into rows of the coarse cell
  if (active) {
    const int Nc = g.N / 2;
    const long long cell = cell_index(Nc, P.lo[0] / 2, P.lo[1] / 2, (D == 3) ? P.lo[2] / 2 : 0);
    T* out = bc + (long long)rhs * ndof_c + cell * NC;
    for (int i = lane; i < NC / n; i += TPP) {
      const int py = i % n, pz = i / n;
      const int base = py * SY + pz * SZ;
      Line<T> v;
      load_line(A, base, 1, v);
#pragma unroll
      for (int nu = 0; nu < n; ++nu) {
        T s = T(0);
#pragma unroll
        for (int p = 0; p < E; ++p) s += T(kRef.P[p * n + nu]) * v.v[p];
        out[i * n + nu] = s;
      }
    }
  }
}

template <typename T, int PPB>
__global__ void __launch_bounds__(TPP * PPB)
k_restrict(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, const T* __restrict__ x,
           const T* __restrict__ b, T* __restrict__ bc, long long ndof, long long ndof_c) {
  __shared__ T smem[PPB * kRestrictPP];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  const int pid = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap) * PPB + slot;
  restrict_body<T>(t, g, scale, x, b, bc, ndof, ndof_c, pid, lane, smem + slot * kRestrictPP, blockIdx.y);
}

// 3-D degrees whose patches span several waves (or do not divide one): the
// same restriction on the register-face operator of k_apply_rf (3-D Q7 in
// FP64, 32^3: 120 us on two tiles, 105 us on its one)
constexpr bool kRestrictOnApplyRF = kApplyRF && !kRestrictRF;
template <typename T, int PPB>
__global__ void __launch_bounds__(TPP * PPB)
k_restrict_rf(const Tab<K, T>* __restrict__ t, PatchGrid g, T scale, const T* __restrict__ x,
              const T* __restrict__ b, T* __restrict__ bc, long long ndof, long long ndof_c) {
  __shared__ T smem[PPB * kApplyRFPP<T>];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  const int pid = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap) * PPB + slot;
  Line<T> xl;
  apply_rf_body<T, RF_RESTRICT>(t, g, scale, x, bc, b, ndof, ndof_c, pid, lane, smem + slot * kApplyRFPP<T>,
                                blockIdx.y, pid < g.npatch, xl);
}

// ------------------------------------------------- prolongation + add
// Where the sums go.  Bound by memory requests: the lines of the last direction
// are read ahead of the contractions and written from registers, n (2-D) or
// n^2 consecutive values a cell, instead of x-rows from the tile after one
// phase and barrier more.  Measured, lines / rows: FP64 3-D Q7 32^3 42.8 / 56.8 us,
// Q6 29.8 / 41.3, Q4 12.3 / 15.5, Q3 7.0 / 8.2, 2-D Q5 256^2 8.4 / 10.3; FP32 3-D Q7
// 22.3 / 24.5, Q3 5.1 / 5.2, 2-D Q7 256^2 7.7 / 8.3.  The rows stay for 3-D Q1 (7.4 /
// 7.1 us on 64^3) and the FP32 lines of short cells (2-D Q6 9.5 / 7.5, Q3 4.4 / 3.9;
// 3-D Q2 64^3 14.8 / 13.2): four-byte pieces of runs of 24 bytes or so cost more
// requests than a row's wide ones.
template <typename T>
constexpr bool kProlongLines = sizeof(T) == 8 ? !(D == 3 && K == 1) : (D == 3 ? K >= 3 : K == 7);

template <typename T>
__device__ __forceinline__ void prolong_body(const PatchGrid& g, const T* __restrict__ xc, T* __restrict__ x,
                                             long long ndof, long long ndof_c, int pid, int lane, T* tile,
                                             int rhs) {
  const bool active = pid < g.npatch;
  const PatchPos P = patch_pos(g, active ? pid : 0);
  const long long roff = (long long)rhs * ndof;
  // This lane's line along the last direction, in 3-D with the lanes cell by
  // cell: n^2 consecutive values a cell.  Its values of x are read ahead of the
  // contractions, and the last pass adds to them and writes them back.
  const int ll = (D == 3) ? (lane / (n * n)) % 2 * n + lane % n + E * (lane / (2 * n * n) * n + lane / n % n) : lane;
  const long long cs = (long long)((D == 3) ? g.N * g.N : g.N) * NC;  // next cell along it
  constexpr int ns = (D == 3) ? n * n : n;
  T* xl = x + roff + node_offset(g.N, P, ll % E, ll / E, 0);
  T xv[E];
  if (kProlongLines<T> && active) {
#pragma unroll
    for (int p = 0; p < E; ++p) xv[p] = xl[(p / n) * cs + (p % n) * ns];
  }
  // along x: coarse rows (ly, lz) straight from global
  if (active) {
    const int Nc = g.N / 2;
    const long long cell = cell_index(Nc, P.lo[0] / 2, P.lo[1] / 2, (D == 3) ? P.lo[2] / 2 : 0);
    const T* in = xc + (long long)rhs * ndof_c + cell * NC;
    for (int i = lane; i < NC / n; i += TPP) {
      const int py = i % n, pz = i / n;
      const int base = py * SY + pz * SZ;
      T v[n];
#pragma unroll
      for (int nu = 0; nu < n; ++nu) v[nu] = in[i * n + nu];
#pragma unroll
      for (int p = 0; p < E; ++p) {
        T s = T(0);
#pragma unroll
        for (int nu = 0; nu < n; ++nu) s += T(kRef.P[p * n + nu]) * v[nu];
        tile[base + p] = s;
      }
    }
  }
  __syncthreads();
  if constexpr (D == 3) {  // along y: lines (px, pz < n)
    if (active) {
      for (int i = lane; i < E * n; i += TPP) {
        const int base = i % E + i / E * SZ;
        T v[n];
#pragma unroll
        for (int nu = 0; nu < n; ++nu) v[nu] = tile[base + nu * SY];
#pragma unroll
        for (int p = 0; p < E; ++p) {
          T s = T(0);
#pragma unroll
          for (int nu = 0; nu < n; ++nu) s += T(kRef.P[p * n + nu]) * v[nu];
          tile[base + p * SY] = s;
        }
      }
    }
    __syncthreads();
  }
  if (active) {
    int base, stride;
    line_geom(D - 1, ll, base, stride);
    T v[n];
#pragma unroll
    for (int nu = 0; nu < n; ++nu) v[nu] = tile[base + nu * stride];
#pragma unroll
    for (int p = 0; p < E; ++p) {
      T s = T(0);
#pragma unroll
      for (int nu = 0; nu < n; ++nu) s += T(kRef.P[p * n + nu]) * v[nu];
      if constexpr (kProlongLines<T>) xl[(p / n) * cs + (p % n) * ns] = xv[p] + s;
      else tile[base + p * stride] = s;
    }
  }
  if constexpr (!kProlongLines<T>) {
    __syncthreads();
    if (active) {
      const int py = lane % E, pz = lane / E;
      int base, stride;
      line_geom(0, lane, base, stride);
      const long long row0 = roff + xrow_offset(g.N, P, py, pz);
#pragma unroll
      for (int a = 0; a < n; ++a) {
        x[row0 + a] += tile[base + a];
        x[row0 + NC + a] += tile[base + n + a];
      }
    }
  }
}

template <typename T, int PPB>
__global__ void __launch_bounds__(TPP * PPB)
k_prolong(const Tab<K, T>* __restrict__ t, PatchGrid g, const T* __restrict__ xc,
          T* __restrict__ x, long long ndof, long long ndof_c) {
  __shared__ T smem[PPB * TS];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  const int pid = xcd_block(blockIdx.x, gridDim.x, g.xcd_remap) * PPB + slot;
  (void)t;
  prolong_body<T>(g, xc, x, ndof, ndof_c, pid, lane, smem + slot * TS, blockIdx.y);
}

// ---------------------------------------------------------- coarse solve
// Level 0 (N = 2): one patch, every node kept (type 3 in all directions).
// Every thread of the workgroup calls this (barriers inside); only threads
// with active set work.
template <typename T>
__device__ __forceinline__ void coarse_body(const Tab<K, T>* __restrict__ t, T inv_scale,
                                            const T* __restrict__ b, T* __restrict__ x, long long ndof,
                                            int lane, T* tile, int rhs, bool active) {
  PatchPos P;
#pragma unroll
  for (int i = 0; i < 3; ++i) { P.lo[i] = 0; P.ty[i] = 3; }
  const long long roff = (long long)rhs * ndof;
  const int nl = active ? NL : 0;  // lines this thread's patch slot works on
  // S_x^T straight from the rows of b
  for (int i = lane; i < nl; i += TPP) {
    const int py = i % E, pz = i / E;
    int base, stride;
    line_geom(0, i, base, stride);
    Line<T> v, o;
    read_xline<T>(b + roff, xrow_offset(2, P, py, pz), v);
    line_St_t<T, 3, SP_DIR>(t, v, o);
    store_line(tile, base, stride, o);
  }
  __syncthreads();
  // S^T along the remaining directions; the last one also scales and applies S
#pragma unroll
  for (int dir = 1; dir < D; ++dir) {
    for (int i = lane; i < nl; i += TPP) {
      int base, stride;
      line_geom(dir, i, base, stride);
      Line<T> v, o;
      load_line(tile, base, stride, v);
      line_St_t<T, 3, SP_DIR>(t, v, o);
      if (dir == D - 1) {
        const int qa = i % E, qb = i / E;
        T lt = t->lam[3][qa];
        if (D == 3) lt += t->lam[3][qb];
#pragma unroll
        for (int q = 0; q < E; ++q) o.v[q] = o.v[q] * (inv_scale * recip(t->lam[3][q] + lt));
        line_S_t<T, 3, SP_DIR>(t, o, v);
        o = v;
      }
      store_line(tile, base, stride, o);
    }
    __syncthreads();
  }
  // S along the directions before the last, ending with x as contiguous rows
#pragma unroll
  for (int dir = D - 2; dir >= 1; --dir) {
    for (int i = lane; i < nl; i += TPP) {
      int base, stride;
      line_geom(dir, i, base, stride);
      Line<T> v, o;
      load_line(tile, base, stride, v);
      line_S_t<T, 3, SP_DIR>(t, v, o);
      store_line(tile, base, stride, o);
    }
    __syncthreads();
  }
  for (int i = lane; i < nl; i += TPP) {
    const int py = i % E, pz = i / E;
    int base, stride;
    line_geom(0, i, base, stride);
    Line<T> v, o;
    load_line(tile, base, stride, v);
    line_S_t<T, 3, SP_DIR>(t, v, o);
    const long long row0 = roff + xrow_offset(2, P, py, pz);
#pragma unroll
    for (int a = 0; a < n; ++a) {
      x[row0 + a] = o.v[a];
      x[row0 + NC + a] = o.v[n + a];
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(TPP)
k_coarse(const Tab<K, T>* __restrict__ t, T inv_scale, const T* __restrict__ b, T* __restrict__ x,
         long long ndof) {
  __shared__ T tile[TS];
  coarse_body<T>(t, inv_scale, b, x, ndof, threadIdx.x, tile, blockIdx.y, true);
}

// ------------------------------------------------------- V-cycle bottom
// Levels 1 (N = 4) and 0 (N = 2) of the V-cycle in one workgroup per
// right-hand side.  A colour of level 1 has at most 2^D patches, one patch
// slot each, so colours follow each other at a barrier instead of a launch:
// pre-smoothing from x = 0 (colours ascending), residual + restriction, the
// exact coarse solve, prolongation + add, post-smoothing (descending).  Every
// patch does the arithmetic of the separate kernels.  In-place smoothers only.
constexpr int kBottomSlots = 1 << D;
constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
constexpr int kBottomPP = max3(kRestrictPP, smooth_pp<1>(), smooth_pp<4>());

template <typename T>
constexpr bool bottom_fits() {
  return TPP * kBottomSlots <= 1024 && kBottomSlots * kBottomPP * (int)sizeof(T) <= 160 * 1024;
}

// the patches of one colour on the level with N cells per direction
__device__ __forceinline__ PatchGrid level_colour(int N, int colour) {
  PatchGrid g{};
  g.N = N;
  g.xcd_remap = 0;
  g.npatch = 1;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int bit = (i < D) ? (colour >> i) & 1 : 0;
    g.off[i] = bit;
    g.cnt[i] = (i < D) ? (bit ? (N - 2) / 2 : N / 2) : 1;
    g.npatch *= g.cnt[i];
  }
  return g;
}
__device__ __forceinline__ PatchGrid level1_colour(int colour) { return level_colour(4, colour); }

template <typename T>
struct BottomArgs {
  T scale1, inv_scale1, scale0_inv;
  T* x1;
  const T* b1;
  T* b0;
  T* x0;
  long long ndof1, ndof0;
};

// the stages of levels 1 and 0 (patch slot `slot`; slots past a colour's
// patches only meet the barriers)
template <typename T, int MODE>
__device__ __forceinline__ void bottom_body(const Tab<K, T>* __restrict__ t, const BottomArgs<T>& a,
                                            int slot, int lane, T* sm, int rhs) {
  constexpr int NCOL = 1 << D;
  smooth_body<T, MODE, false, true>(t, level1_colour(0), a.scale1, a.inv_scale1, a.x1, a.x1, a.b1,
                                    a.ndof1, slot, lane, sm, rhs);
  __syncthreads();
  for (int c = 1; c < NCOL; ++c) {
    smooth_body<T, MODE, false, false>(t, level1_colour(c), a.scale1, a.inv_scale1, a.x1, a.x1, a.b1,
                                       a.ndof1, slot, lane, sm, rhs);
    __syncthreads();
  }
  restrict_body<T>(t, level1_colour(0), a.scale1, a.x1, a.b1, a.b0, a.ndof1, a.ndof0, slot, lane, sm, rhs);
  __syncthreads();
  coarse_body<T>(t, a.scale0_inv, a.b0, a.x0, a.ndof0, lane, sm, rhs, slot == 0);
  __syncthreads();
  prolong_body<T>(level1_colour(0), a.x0, a.x1, a.ndof1, a.ndof0, slot, lane, sm, rhs);
  __syncthreads();
  for (int c = NCOL - 1; c >= 0; --c) {
    smooth_body<T, MODE, false, false>(t, level1_colour(c), a.scale1, a.inv_scale1, a.x1, a.x1, a.b1,
                                       a.ndof1, slot, lane, sm, rhs);
    __syncthreads();
  }
}

template <typename T, int MODE>
__global__ void __launch_bounds__(TPP * kBottomSlots)
k_bottom(const Tab<K, T>* __restrict__ t, BottomArgs<T> a) {
  __shared__ T smem[kBottomSlots * kBottomPP];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  bottom_body<T, MODE>(t, a, slot, lane, smem + slot * kBottomPP, blockIdx.y);
}

// 2-D: levels 2 (N = 8) to 0 in one workgroup.  A level-2 colour has at most
// 16 patches (16 slots of E threads), so level 2's smoothing, its restriction
// and the prolongation back to it join the stages of levels 1 and 0.  Same
// bodies, so the results equal the separate kernels bit for bit.
constexpr int kBottom3Slots = 16;

template <typename T>
constexpr bool bottom3_fits() {
  return D == 2 && TPP * kBottom3Slots <= 1024 && kBottom3Slots * kBottomPP * (int)sizeof(T) <= 160 * 1024;
}

template <typename T>
struct Bottom3Args {
  BottomArgs<T> a;  // levels 1 and 0 (a.b1 is written here by the level-2 restriction)
  T scale2, inv_scale2;
  T* x2;
  const T* b2;
  T* b1w;
  long long ndof2;
};

template <typename T, int MODE>
__global__ void __launch_bounds__(TPP * kBottom3Slots)
k_bottom3(const Tab<K, T>* __restrict__ t, Bottom3Args<T> a3) {
  __shared__ T smem[kBottom3Slots * kBottomPP];
  const int slot = slot_of(), lane = threadIdx.x % TPP;
  T* sm = smem + slot * kBottomPP;
  const int rhs = blockIdx.y;
  constexpr int NCOL = 1 << D;
  smooth_body<T, MODE, false, true>(t, level_colour(8, 0), a3.scale2, a3.inv_scale2, a3.x2, a3.x2, a3.b2,
                                    a3.ndof2, slot, lane, sm, rhs);
  __syncthreads();
  for (int c = 1; c < NCOL; ++c) {
    smooth_body<T, MODE, false, false>(t, level_colour(8, c), a3.scale2, a3.inv_scale2, a3.x2, a3.x2,
                                       a3.b2, a3.ndof2, slot, lane, sm, rhs);
    __syncthreads();
  }
  restrict_body<T>(t, level_colour(8, 0), a3.scale2, a3.x2, a3.b2, a3.b1w, a3.ndof2, a3.a.ndof1, slot, lane,
                   sm, rhs);
  __syncthreads();
  bottom_body<T, MODE>(t, a3.a, slot, lane, sm, rhs);
  prolong_body<T>(level_colour(8, 0), a3.a.x1, a3.x2, a3.ndof2, a3.a.ndof1, slot, lane, sm, rhs);
  __syncthreads();
  for (int c = NCOL - 1; c >= 0; --c) {
    smooth_body<T, MODE, false, false>(t, level_colour(8, c), a3.scale2, a3.inv_scale2, a3.x2, a3.x2,
                                       a3.b2, a3.ndof2, slot, lane, sm, rhs);
    __syncthreads();
  }
}

// The same with two waves per patch in the smoothing stages (where kSplitOK
// and 2^D two-wave slots fit one workgroup: 3-D Q3): waves 2s and 2s + 1 form
// patch slot s, and the transfer and coarse stages run on the even waves while
// the odd ones meet the barriers only.  The split smoothing body gives every
// output bit for bit as the one-wave body.  Clamped kernel only: the direct form
// is faster with one wave here (V-cycle on 4^3 cells, two waves / one: FP64 119 / 91 us,
// FP32 74 / 66), its halves being code of their own that one workgroup fetches for
// every stage.
constexpr bool kBottomSplitOK = kSplitOK && 2 * TPP * kBottomSlots <= 1024;

template <typename T, int MODE, bool ZERO>
__device__ __forceinline__ void bottom_smooth_half(const Tab<K, T>* __restrict__ t, int colour,
                                                   const BottomArgs<T>& a, int slot, int h, int lane,
                                                   T* sm, int rhs) {
  if (h == 0)
    smooth_split_body<T, MODE, false, ZERO, 0>(t, level1_colour(colour), a.scale1, a.inv_scale1, a.x1,
                                               a.b1, a.ndof1, slot, lane, sm, rhs);
  else
    smooth_split_body<T, MODE, false, ZERO, 1>(t, level1_colour(colour), a.scale1, a.inv_scale1, a.x1,
                                               a.b1, a.ndof1, slot, lane, sm, rhs);
}

template <typename T, int MODE>
__global__ void __launch_bounds__(2 * TPP * kBottomSlots)
k_bottom_split(const Tab<K, T>* __restrict__ t, BottomArgs<T> a) {
  static_assert(kBottomSplitOK, "two-wave slots must fit one workgroup");
  __shared__ T smem[kBottomSlots * kBottomPP];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TPP);
  const int slot = w / 2, h = w % 2, lane = threadIdx.x % TPP;
  const int tslot = h == 0 ? slot : kBottomSlots;  // one-wave stages: odd waves hold no patch
  T* sm = smem + slot * kBottomPP;
  const int rhs = blockIdx.y;
  constexpr int NCOL = 1 << D;
  bottom_smooth_half<T, MODE, true>(t, 0, a, slot, h, lane, sm, rhs);
  __syncthreads();
  for (int c = 1; c < NCOL; ++c) {
    bottom_smooth_half<T, MODE, false>(t, c, a, slot, h, lane, sm, rhs);
    __syncthreads();
  }
  restrict_body<T>(t, level1_colour(0), a.scale1, a.x1, a.b1, a.b0, a.ndof1, a.ndof0, tslot, lane, sm, rhs);
  __syncthreads();
  coarse_body<T>(t, a.scale0_inv, a.b0, a.x0, a.ndof0, lane, sm, rhs, slot == 0 && h == 0);
  __syncthreads();
  prolong_body<T>(level1_colour(0), a.x0, a.x1, a.ndof1, a.ndof0, tslot, lane, sm, rhs);
  __syncthreads();
  for (int c = NCOL - 1; c >= 0; --c) {
    bottom_smooth_half<T, MODE, false>(t, c, a, slot, h, lane, sm, rhs);
    __syncthreads();
  }
}

// ------------------------------------------------------------ launchers
// Workgroup shapes the autotuner chooses between: PPB_DEFAULT patches per
// workgroup (variant 0) or twice as many (variant 1) while the workgroup stays
// within 256 threads (larger patches keep one per workgroup).
template <int V>
struct Shape {
  static constexpr int PPB =
      (V == 1 && TPP * PPB_DEFAULT * 2 > 256) ? PPB_DEFAULT : PPB_DEFAULT * (V + 1);
};

// Slots of the right-hand-side-packed shapes: at most 8 (3-D) or 16 (2-D)
// per workgroup, within 1024 threads and half the LDS of a CU.
template <typename T, int PP>
constexpr int rpack_slots() {
  int r = (D == 3) ? 8 : 16;
  while (r > 1 && (TPP * r > 1024 || r * PP * (int)sizeof(T) > kPackedLDS)) r /= 2;
  return r;
}
template <typename T>
constexpr int rpack_apply_slots() {
  return kApplyRF ? rpack_slots<T, kApplyRFPP<T>>()
                  : rpack_slots<T, Smem<2, (D - 1) * 2 * 2 * NF>::per_patch>();
}

template <typename T, int V>
hipError_t launch_apply(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                        long long ndof, hipStream_t s) {
  constexpr int PPB = Shape<V>::PPB;
  g.nrhs = nrhs;
  dim3 grid((g.npatch + PPB - 1) / PPB, nrhs);
  hipLaunchKernelGGL((k_apply<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                     (const Tab<K, T>*)tab, g, scale, x, y, ndof);
  return hipGetLastError();
}
// shape 2: face data in registers where kApplyRF (otherwise shape 0)
template <typename T>
hipError_t launch_apply_rf(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                           long long ndof, hipStream_t s) {
  if constexpr (!kApplyRF) {
    return launch_apply<T, 0>(tab, g, scale, x, y, nrhs, ndof, s);
  } else {
    constexpr int PPB = PPB_DEFAULT;
    g.nrhs = nrhs;
    dim3 grid((g.npatch + PPB - 1) / PPB, nrhs);
    hipLaunchKernelGGL((k_apply_rf<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                       (const Tab<K, T>*)tab, g, scale, x, y, ndof);
    return hipGetLastError();
  }
}
// shape 3: one patch for several right-hand sides per workgroup (face data
// in registers in 3-D)
template <typename T>
hipError_t launch_apply_rpack(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                              long long ndof, hipStream_t s) {
  constexpr int R = rpack_apply_slots<T>();
  g.nrhs = nrhs;
  const dim3 grid(g.npatch, (nrhs + R - 1) / R), block(TPP * R);
  if constexpr (kApplyRF)
    hipLaunchKernelGGL((k_apply_rf<T, R, true>), grid, block, 0, s, (const Tab<K, T>*)tab, g, scale, x, y,
                       ndof);
  else
    hipLaunchKernelGGL((k_apply<T, R, true>), grid, block, 0, s, (const Tab<K, T>*)tab, g, scale, x, y,
                       ndof);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_mass(const void* tab, PatchGrid g, T scale, const T* x, T* y, int nrhs,
                       long long ndof, hipStream_t s) {
  constexpr int PPB = PPB_DEFAULT;
  dim3 grid((g.npatch + PPB - 1) / PPB, nrhs);
  hipLaunchKernelGGL((k_mass<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                     (const Tab<K, T>*)tab, g, scale, x, y, ndof);
  return hipGetLastError();
}
// smoother shapes: bit 0 selects the workgroup shape, bit 1 the prefetch of b
// (not in the direct form, which has one order of loads), bit 2 two waves per
// patch where kSplitOK (not the Full kernel), else one patch per workgroup where
// several patches share a wave (2-D, 3-D Q1: patches of different types there run
// their fast-diagonalisation branches one after the other), else the same as
// bit 2 clear; variant 0 / 1 / 2 / 3: Dirichlet consistent / Dirichlet with
// the paper's residual / Full / clamped
constexpr bool kOnePatchShape = !kSplitOK && PPB_DEFAULT > 1;
// shapes 8..11 (bit 3): one patch for several right-hand sides per workgroup,
// bit 0 selecting the larger slot count (by the variant's own LDS footprint),
// bit 1 the prefetch of b
template <typename T, int MODE>
constexpr int rpack_smooth_slots(bool large) {
  constexpr int r = rpack_slots<T, smooth_pp<MODE, T>()>();
  return large ? r : (r > 1 ? r / 2 : 1);
}
template <typename T, int MODE, bool LARGE, bool PF>
hipError_t launch_smooth_rpack(const Tab<K, T>* tb, PatchGrid g, T scale, T inv_scale, int zero, const T* xin,
                               T* xout, const T* b, int nrhs, long long ndof, hipStream_t s) {
  constexpr int R = rpack_smooth_slots<T, MODE>(LARGE);
  constexpr bool PFD = PF && !kDirect<MODE>;
  const dim3 grid(g.npatch, (nrhs + R - 1) / R), block(TPP * R);
  if (zero)
    hipLaunchKernelGGL((k_smooth<T, R, MODE, false, true, true>), grid, block, 0, s, tb, g, scale, inv_scale, xin,
                       xout, b, ndof);
  else if (kDirect<MODE> && g.guard)
    hipLaunchKernelGGL((k_smooth<T, R, MODE, PFD, false, true, kDirect<MODE>>), grid, block, 0, s, tb, g, scale,
                       inv_scale, xin, xout, b, ndof);
  else
    hipLaunchKernelGGL((k_smooth<T, R, MODE, PFD, false, true>), grid, block, 0, s, tb, g, scale, inv_scale, xin,
                       xout, b, ndof);
  return hipGetLastError();
}
template <typename T, int PPB, int MODE, bool PF>
hipError_t launch_smooth_split(const Tab<K, T>* tb, PatchGrid g, T scale, T inv_scale, int zero, T* x, const T* b,
                               int nrhs, long long ndof, hipStream_t s) {
  constexpr bool PFD = PF && !kDirect<MODE>;
  const dim3 grid((g.npatch + PPB - 1) / PPB, nrhs), block(2 * TPP * PPB);
  if (zero)
    hipLaunchKernelGGL((k_smooth_split<T, PPB, MODE, false, true>), grid, block, 0, s, tb, g, scale, inv_scale, x, b,
                       ndof);
  else if (kDirect<MODE> && g.guard)
    hipLaunchKernelGGL((k_smooth_split<T, PPB, MODE, PFD, false, kDirect<MODE>>), grid, block, 0, s, tb, g, scale,
                       inv_scale, x, b, ndof);
  else
    hipLaunchKernelGGL((k_smooth_split<T, PPB, MODE, PFD>), grid, block, 0, s, tb, g, scale, inv_scale, x, b, ndof);
  return hipGetLastError();
}
template <typename T, int PPB, int MODE, bool PF>
hipError_t launch_smooth_patches(const Tab<K, T>* tb, PatchGrid g, T scale, T inv_scale, int zero, const T* xin,
                                 T* xout, const T* b, int nrhs, long long ndof, hipStream_t s) {
  constexpr bool PFD = PF && !kDirect<MODE>;
  const dim3 grid((g.npatch + PPB - 1) / PPB, nrhs), block(TPP * PPB);
  if (zero)  // x = 0, colour 0: the residual is b, no prefetch needed
    hipLaunchKernelGGL((k_smooth<T, PPB, MODE, false, true>), grid, block, 0, s, tb, g, scale, inv_scale, xin, xout,
                       b, ndof);
  else if (kDirect<MODE> && g.guard)
    hipLaunchKernelGGL((k_smooth<T, PPB, MODE, PFD, false, false, kDirect<MODE>>), grid, block, 0, s, tb, g, scale,
                       inv_scale, xin, xout, b, ndof);
  else
    hipLaunchKernelGGL((k_smooth<T, PPB, MODE, PFD>), grid, block, 0, s, tb, g, scale, inv_scale, xin, xout, b, ndof);
  return hipGetLastError();
}
// shape V of one kernel
template <typename T, int V, int MODE>
hipError_t launch_smooth_mode(const Tab<K, T>* tb, PatchGrid g, T scale, T inv_scale, int zero, const T* xin, T* xout,
                              const T* b, int nrhs, long long ndof, hipStream_t s) {
  constexpr int PPB = (kOnePatchShape && (V & 4)) ? 1 : Shape<(V & 1)>::PPB;
  constexpr bool PF = (V & 2) != 0;
  if constexpr ((V & 8) != 0)
    return launch_smooth_rpack<T, MODE, (V & 1) != 0, PF>(tb, g, scale, inv_scale, zero, xin, xout, b, nrhs, ndof, s);
  else if constexpr ((V & 4) != 0 && kSplitOK && MODE != 3)
    return launch_smooth_split<T, PPB, MODE, PF>(tb, g, scale, inv_scale, zero, xout, b, nrhs, ndof, s);
  else
    return launch_smooth_patches<T, PPB, MODE, PF>(tb, g, scale, inv_scale, zero, xin, xout, b, nrhs, ndof, s);
}
template <typename T, int V>
hipError_t launch_smooth(const void* tab, PatchGrid g, T scale, T inv_scale, int variant, int zero,
                         const T* xin, T* xout, const T* b, int nrhs, long long ndof, hipStream_t s) {
  g.nrhs = nrhs;
  const Tab<K, T>* tb = (const Tab<K, T>*)tab;
  if (variant == 2)
    return launch_smooth_mode<T, V, 3>(tb, g, scale, inv_scale, zero, xin, xout, b, nrhs, ndof, s);
  if (variant == 3)
    return launch_smooth_mode<T, V, 4>(tb, g, scale, inv_scale, zero, xout, xout, b, nrhs, ndof, s);
  if constexpr (kBothForms<T>) {
    if (g.N >= direct_below(D, K, sizeof(T))) {
      if (variant == 1)
        return launch_smooth_mode<T, V, 6>(tb, g, scale, inv_scale, zero, xout, xout, b, nrhs, ndof, s);
      return launch_smooth_mode<T, V, 5>(tb, g, scale, inv_scale, zero, xout, xout, b, nrhs, ndof, s);
    }
  }
  if (variant == 1)
    return launch_smooth_mode<T, V, 2>(tb, g, scale, inv_scale, zero, xout, xout, b, nrhs, ndof, s);
  return launch_smooth_mode<T, V, 1>(tb, g, scale, inv_scale, zero, xout, xout, b, nrhs, ndof, s);
}
template <typename T>
hipError_t launch_restrict(const void* tab, PatchGrid g, T scale, const T* x, const T* b, T* bc,
                           int nrhs, long long ndof, long long ndof_c, hipStream_t s) {
  constexpr int PPB = PPB_DEFAULT;
  dim3 grid((g.npatch + PPB - 1) / PPB, nrhs);
  if constexpr (kRestrictOnApplyRF)
    hipLaunchKernelGGL((k_restrict_rf<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                       (const Tab<K, T>*)tab, g, scale, x, b, bc, ndof, ndof_c);
  else
    hipLaunchKernelGGL((k_restrict<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                       (const Tab<K, T>*)tab, g, scale, x, b, bc, ndof, ndof_c);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_prolong(const void* tab, PatchGrid g, const T* xc, T* x, int nrhs,
                          long long ndof, long long ndof_c, hipStream_t s) {
  constexpr int PPB = PPB_DEFAULT;
  dim3 grid((g.npatch + PPB - 1) / PPB, nrhs);
  hipLaunchKernelGGL((k_prolong<T, PPB>), grid, dim3(TPP * PPB), 0, s,
                     (const Tab<K, T>*)tab, g, xc, x, ndof, ndof_c);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_coarse(const void* tab, T inv_scale, const T* b, T* x, int nrhs, long long ndof,
                         hipStream_t s) {
  dim3 grid(1, nrhs);
  hipLaunchKernelGGL((k_coarse<T>), grid, dim3(TPP), 0, s, (const Tab<K, T>*)tab, inv_scale, b, x,
                     ndof);
  return hipGetLastError();
}

// variant 0 / 1 / 3 (in-place smoothers); the Full kernel is not fused.
// split: two waves per patch in the smoothing stages where kBottomSplitOK.
template <typename T>
hipError_t launch_bottom(const void* tab, int variant, int split, T scale1, T inv_scale1, T inv_scale0,
                         T* x1, const T* b1, T* b0, T* x0, int nrhs, long long ndof1, long long ndof0,
                         hipStream_t s) {
  if constexpr (!bottom_fits<T>()) {
    return hipErrorInvalidConfiguration;
  } else {
    const BottomArgs<T> a{scale1, inv_scale1, inv_scale0, x1, b1, b0, x0, ndof1, ndof0};
    const Tab<K, T>* tb = (const Tab<K, T>*)tab;
    const dim3 grid(1, nrhs), block(TPP * kBottomSlots);
    if constexpr (kBottomSplitOK) {
      if (split && variant == 3) {
        hipLaunchKernelGGL((k_bottom_split<T, 4>), grid, dim3(2 * TPP * kBottomSlots), 0, s, tb, a);
        return hipGetLastError();
      }
    }
    if (variant == 0) hipLaunchKernelGGL((k_bottom<T, 1>), grid, block, 0, s, tb, a);
    else if (variant == 1) hipLaunchKernelGGL((k_bottom<T, 2>), grid, block, 0, s, tb, a);
    else if (variant == 3) hipLaunchKernelGGL((k_bottom<T, 4>), grid, block, 0, s, tb, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
}

// levels 2, 1, 0 in one launch (2-D; variants 0 / 1 / 3)
template <typename T>
hipError_t launch_bottom3(const void* tab, int variant, T scale2, T inv_scale2, T scale1, T inv_scale1,
                          T inv_scale0, T* x2, const T* b2, T* x1, T* b1, T* b0, T* x0, int nrhs,
                          long long ndof2, long long ndof1, long long ndof0, hipStream_t s) {
  if constexpr (!bottom3_fits<T>()) {
    return hipErrorInvalidConfiguration;
  } else {
    Bottom3Args<T> a3;
    a3.a = BottomArgs<T>{scale1, inv_scale1, inv_scale0, x1, b1, b0, x0, ndof1, ndof0};
    a3.scale2 = scale2;
    a3.inv_scale2 = inv_scale2;
    a3.x2 = x2;
    a3.b2 = b2;
    a3.b1w = b1;
    a3.ndof2 = ndof2;
    const Tab<K, T>* tb = (const Tab<K, T>*)tab;
    const dim3 grid(1, nrhs), block(TPP * kBottom3Slots);
    if (variant == 0) hipLaunchKernelGGL((k_bottom3<T, 1>), grid, block, 0, s, tb, a3);
    else if (variant == 1) hipLaunchKernelGGL((k_bottom3<T, 2>), grid, block, 0, s, tb, a3);
    else if (variant == 3) hipLaunchKernelGGL((k_bottom3<T, 4>), grid, block, 0, s, tb, a3);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
}

template <typename T>
KernelSet<T> make_set() {
  KernelSet<T> k;
  k.apply[0] = &launch_apply<T, 0>;
  k.apply[1] = &launch_apply<T, 1>;
  k.apply[2] = &launch_apply_rf<T>;
  k.apply[3] = &launch_apply_rpack<T>;
  k.two_counts = Shape<1>::PPB != Shape<0>::PPB ? 1 : 0;
  k.one_patch = kOnePatchShape ? 1 : 0;
  k.apply_rf = kApplyRF ? 1 : 0;
  k.apply_rpack = rpack_apply_slots<T>() > 1 ? 1 : 0;
  k.smooth_rpack[0] = rpack_smooth_slots<T, 1>(true);
  k.smooth_rpack[1] = rpack_smooth_slots<T, 2>(true);
  k.smooth_rpack[2] = rpack_smooth_slots<T, 3>(true);
  k.smooth_rpack[3] = rpack_smooth_slots<T, 4>(true);
  k.mass = &launch_mass<T>;
  k.smooth[0] = &launch_smooth<T, 0>;
  k.smooth[1] = &launch_smooth<T, 1>;
  k.smooth[2] = &launch_smooth<T, 2>;
  k.smooth[3] = &launch_smooth<T, 3>;
  k.smooth[4] = &launch_smooth<T, 4>;
  k.smooth[5] = &launch_smooth<T, 5>;
  k.smooth[6] = &launch_smooth<T, 6>;
  k.smooth[7] = &launch_smooth<T, 7>;
  k.smooth[8] = &launch_smooth<T, 8>;
  k.smooth[9] = &launch_smooth<T, 9>;
  k.smooth[10] = &launch_smooth<T, 10>;
  k.smooth[11] = &launch_smooth<T, 11>;
  k.smooth_split = kSplitOK ? 1 : 0;
  k.direct_below = kDirect<1> ? direct_below(D, K, sizeof(T)) : 0;
  k.restrict_residual = &launch_restrict<T>;
  k.prolongate_add = &launch_prolong<T>;
  k.coarse = &launch_coarse<T>;
  k.bottom = bottom_fits<T>() ? &launch_bottom<T> : nullptr;
  k.bottom_split = (bottom_fits<T>() && kBottomSplitOK) ? 1 : 0;
  k.bottom3 = bottom3_fits<T>() ? &launch_bottom3<T> : nullptr;
  return k;
}

}  // namespace
}  // namespace dgmg

#define DGMG_CAT2(a, b, c, d) a##b##c##d
#define DGMG_ENTRY(Dv, Kv) DGMG_CAT2(dgmg_kernels_d, Dv, _k, Kv)
extern "C" void DGMG_ENTRY(DGMG_D, DGMG_K)(dgmg::KernelEntry* e) {
  e->dim = DGMG_D;
  e->degree = DGMG_K;
  e->f64 = dgmg::make_set<double>();
  e->f32 = dgmg::make_set<float>();
}

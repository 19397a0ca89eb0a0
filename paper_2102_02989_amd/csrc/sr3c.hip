// sr3c.hip -- short-range (erfc-attenuated) three-center lattice sums on gfx950.
//
// Work item: (aux shell P, AO shell pair); a wavefront takes a range of BvK
// cells c1 and an interleaved share of the pair images (SRWork).
// The term (P^0 | erfc(w r)/r | mu^m nu^{m+n'}) of Eq. (M12)/(M13a) is
// rewritten by translation as (P^{-m} | mu^0 nu^{n'}): for a pair image n' the
// AO pair density is fixed and the aux function moves over lattice vectors m.
// Terms are grouped by Born-von Karman cells (Eq. M14): c1 = c(m) and
// c2 = c(m + n').
//
// Lane layout: a lane takes one unit, that is a pair image n', a BvK cell c1 and a
// share of the lattice vectors m of that cell; a wave takes rows of ncb cells,
// a row being (a share of) an image, and images in the pair list order (sorted
// by the BvK class of n', so the target (c1, c2) changes only with the class).
//   1. 64 images at a time are put to the per-term window test of the
//      Supplementary Material (Eqs. S23-S25, most diffuse primitives as 1s
//      functions); the kept ones queue up in LDS, and a batch of them gets the
//      wave's rows in proportion to its lattice vectors;
//   2. every lane lists the lattice vectors of its unit inside the screening
//      radius (R_c <= R_c^cut of Eq. S14 and R12 <= R12^cut(R_c));
//   3. for every primitive triple it sums the Hermite Coulomb integrals R_tuv of
//      the erfc operator over its list (the only m-dependent factor of the
//      McMurchie-Davidson expression) and contracts them with the pair's E^ab,
//      in its registers (or, for the classes with the most components, through
//      LDS with a lane per (cell, aux Hermite order));
//   4. when the class of n' ends, the lanes are added in row order, the aux
//      coefficients E^c applied, and X[c1][c2][P][mu][nu] (or the wave's partial
//      block when the images of the item are split over several waves) stored.
// Every X element (and every partial element) is owned by one wave and stored
// once, so results are deterministic without atomics; split items are summed
// by sr_reduce_kernel in slice order.
#include <hip/hip_runtime.h>

#include "boys.h"
#include "device_math.h"
#include "kernels.h"
#include "lanes.h"
#include "plan.h"

namespace rsgdf {

constexpr int kSRWinCap = 256;    // screening windows held in LDS
constexpr int kTripC = 9;         // constants per primitive triple

// Constants of a primitive triple (AO a, AO b, aux c) that do not depend on
// the pair image: t[0] 1/p, t[1] g_b/p (P = A + t[1] (B - A)), t[2] g_a g_b/p
// (K_ab = e^{-t[2] R12^2}), t[3] rho, t[4] theta^2, t[5] theta, t[6] the
// signed contraction prefactor c_c c_a c_b 2 pi^{5/2}/(p g_c sqrt(p + g_c)),
// t[7] the 1s screening estimate per unit K_ab and lattice vector
// (Eqs. S4-S9 with the erfc attenuation), t[8] 1/(2 g_c).
template <int LP>
__device__ __forceinline__ void triple_consts(double ga, double gb, double gc, double ca, double cb, double cc,
                                              double ca1, double cb1, double cc1, double omega, double acut,
                                              double *t) {
  const double p = ga + gb, oop = 1.0 / p;
  const double rpc = 1.0 / (p + gc);
  const double rho = p * gc * rpc;
  const double om2 = omega * omega;
  const double th2 = om2 / (om2 + rho);
  const double e1 = sqrt(rho);
  const double e2 = 1.0 / sqrt(1.0 / rho + 1.0 / om2);
  t[0] = oop;
  t[1] = gb * oop;
  t[2] = ga * gb * oop;
  t[3] = rho;
  t[4] = th2;
  t[5] = sqrt(th2);
  t[6] = ((LP & 1) ? -1.0 : 1.0) * cc * ca * cb * 2.0 * kPi * kPi * sqrt(kPi) * sqrt(rpc) / (p * gc);
  t[7] = kPi * kPi * kPi * cc1 * ca1 * cb1 / (gc * p * sqrt(gc * p)) * 2.0 * (e1 - e2) *
         0.564189583547756286948079451561;
  t[8] = 0.5 / gc;
  // compact/diffuse split: a diffuse aux primitive or two diffuse AO
  // primitives put the triple into the Eq. M15 part; a zero screening estimate
  // makes the image loop's primitive screen skip it
  if (acut > 0.0 && (gc < acut || (ga < acut && gb < acut))) {
    t[6] = 0.0;
    t[7] = 0.0;
  }
}


__device__ __forceinline__ int pack3(int a, int b, int c) {
  return ((a + 512) & 1023) | (((b + 512) & 1023) << 10) | (((c + 512) & 1023) << 20);
}
__device__ __forceinline__ void unpack3(int v, int &a, int &b, int &c) {
  a = (v & 1023) - 512;
  b = ((v >> 10) & 1023) - 512;
  c = ((v >> 20) & 1023) - 512;
}

// ---- one unit per lane ----------------------------------------------------------
// Powers of Cartesian component n of angular momentum l (x descending, then y).
__host__ __device__ constexpr int crt_r(int n) { return (n >= 1) + (n >= 3) + (n >= 6); }
__host__ __device__ constexpr int crt_x(int l, int n) { return l - crt_r(n); }
__host__ __device__ constexpr int crt_z(int, int n) { return n - crt_r(n) * (crt_r(n) + 1) / 2; }
__host__ __device__ constexpr int crt_y(int l, int n) { return l - crt_x(l, n) - crt_z(l, n); }
// power of axis d of aux Hermite order i of a shell LP (|tau| = LP, then LP - 2)
__host__ __device__ constexpr int tau_pow(int LP, int i, int d) {
  const int l = i < ncart(LP) ? LP : LP - 2, n = i < ncart(LP) ? i : i - ncart(LP);
  return d == 0 ? crt_x(l, n) : (d == 1 ? crt_y(l, n) : crt_z(l, n));
}
// index of aux component ic lowered by two in axis d among the components of LP - 2
__host__ __device__ constexpr int tau_low(int LP, int ic, int d) {
  const int x = crt_x(LP, ic) - (d == 0 ? 2 : 0), z = crt_z(LP, ic) - (d == 2 ? 2 : 0);
  const int r = LP - 2 - x;
  return r * (r + 1) / 2 + z;
}

// f(integral constant i) for i = 0 .. N - 1: every index of the register arrays
// below stays a constant (the unroller leaves the larger classes' loops rolled
// and their arrays in scratch memory)
template <int I>
struct IntC {
  static constexpr int v = I;
};
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(IntC<I>{});
    static_for<I + 1, N>(f);
  }
}

constexpr int kUnitQueue = 128; // pair images waiting in LDS
constexpr int kUnitFl = 6;      // components per step of the flush
constexpr int kUnitTrip = 20;   // primitive triples whose constants are held in LDS
constexpr int kUnitWaves = 4;   // waves per workgroup (they share the Boys table and nothing else)

// item constants in LDS: centres A, B, C; window test; diffuse pair centre
// A + t1d (B - A); reciprocal rows / 2 pi, their norms, reciprocal mesh
enum { uA = 0, uB = 3, uC = 6, uBeta = 9, uXstar, uGmax, uGrow, uR12min, uRc, uT1d, uRb, uSp = uRb + 9, uOn = uSp + 3,
       uNum = uOn + 3 };
enum { nPa = 0, nPb, nPp, nTa, nTb, nTp, nFa, nFb, nFp, nDiag, nMesh, nNcb = nMesh + 3, nImg, nCoff, nNsr, nW, nNum };
// the classes with more accumulators than a lane holds
constexpr int kWideUnits = 16;  // units whose Hermite sums are in LDS at a time
constexpr int kWideRows = 8;    // most rows (images) among them
// offset of E^{ij}_t, t = 0 .. i + j, in a row of the nonzero coefficients (i, then j)
__host__ __device__ constexpr int e_off(int LB, int i, int j) {
  int o = 0;
  for (int a = 0; a <= i; ++a)
    for (int b = 0; b <= (a == i ? j - 1 : LB); ++b) o += a + b + 1;
  return o;
}
// powers of Hermite index h (inverse of hidx)
__host__ __device__ constexpr int herm_pow(int h, int d) {
  int s = 0;
  while (nherm(s) <= h) ++s;
  const int rem = h - (s > 0 ? nherm(s - 1) : 0);
  int r = 0;
  while ((r + 1) * (r + 2) / 2 <= rem) ++r;
  const int v = rem - r * (r + 1) / 2;
  return d == 0 ? s - r : (d == 1 ? r - v : v);
}
constexpr int kUnitClsBits = 20, kUnitClsMask = (1 << kUnitClsBits) - 1;

// LDS written by some lanes of the wave is read by others: program order of the
// wave's own LDS accesses is enough, the compiler has to keep it
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// waves per SIMD by the doubles a lane keeps live (Hermite sums, recursion
// scratch, accumulators)
__host__ __device__ constexpr int sr_unit_waves(int LP, int LA, int LB) {
  const int L = LP + LA + LB;
  const int d = nherm(L) + (L > 0 ? nherm(L - 1) : 0) +
                (sr_unit_class(LP, LA, LB) ? sr_ntau(LP) : 2) * ncart(LA) * ncart(LB);
  return d <= 30 ? 3 : (d <= 75 ? 2 : 1);
}

// Lattice vectors that a lane lists, and contracts at once: as many as leave the
// workgroups that the registers allow their LDS (one of 108 to 159 KB per CU where a
// lane has the registers of a SIMD to itself, else two of 76 KB).  With 12 in every class
// the contractions, one per pass, were the work where a unit has hundreds of vectors:
// 8 atoms 2x2x2, omega 0.1: 3370 ms of short range, 2570 with these.
__host__ __device__ constexpr int sr_unit_cand(int LP, int LA, int LB) {
  if (sr_unit_waves(LP, LA, LB) > 1 || LP + LA + LB == 7) return 32;
  return sr_unit_class(LP, LA, LB) ? 64 : 48;
}
// Vectors per lane at which a batch of images is full: more where a contraction costs
// more.  (With 12 per pass 4, 6 and 10 took 153, 149 and 143 ms for 8 atoms 2x2x2 and
// 198, 180 and 175 for 5 atoms 2x2x1: a batch's set-up outweighs its even lanes.)
__host__ __device__ constexpr int sr_unit_fill(int LP, int LA, int LB) {
  return sr_unit_waves(LP, LA, LB) > 1 ? 10 : 24;
}

// A lane takes one unit: a pair image n', a BvK cell c1 and a share of the
// lattice vectors m of that cell.  It sums the Hermite integrals of its
// vectors in registers, contracts them with the pair's E^ab there, and keeps
// the sums over (aux Hermite order tau, AO components) in registers for all
// primitive triples and all batches of images of one BvK class; only then are
// the lanes added up through LDS (row order) and stored.  No reduction, no
// barrier and no table of indices inside the loop over primitive triples.
// The aux coefficients are applied at the store: for a single centre
//   prod_d E^{c_d}_{tau_d} = (1/2g)^{(lP + |tau|)/2} kappa,
// kappa = 1 for tau = c, and 1 (c_d = 2) or 3 (c_d = 3) for tau = c - 2 e_d,
// so the exponent enters as a factor of the contraction and kappa at the end.
//
// What bounds it: FP64 issue and the lanes that run out of lattice vectors
// before their wave does (about half of the lanes are active per instruction
// where an image has 2 to 6 vectors per cell).  The registers decide the rest:
// with the item's constants in registers every class spilled 200 to 700 bytes
// per lane and waited for scratch memory 40-65% of its cycles; in LDS they
// leave no class up to 75 live doubles with more than 20 bytes.  Against the
// wave-cooperative kernel below 126 accumulators (short-range phase): 8 atoms
// double zeta 2x2x2, omega 0.5: 692 -> 238 ms; 4 atoms 3x3x3, omega 1.5: 646 ->
// 167 ms; 3 atoms 1x3x2, omega 1: 247 -> 94 ms; 12 atoms single zeta 4x4x4,
// omega 0.1: 274 -> 89 ms; 2 atoms at Gamma, omega 0.1: 1.51 -> 1.2 ms.
//
// The wide classes ((d|dd), (f|dp), (f|dd)) would need 234 to 468 accumulators a
// lane.  Their sums cross LDS: 16 units at a time, whose R_tuv the lanes of
// (cell, tau) gather at h + tau, each keeping its NAB components in registers.
// With the cooperative kernel for these three the first three workloads above
// were 238, 167 and 94 ms; they are 139, 101 and 37 ms.
template <int LP, int LA, int LB>
__global__ __launch_bounds__(64 * kUnitWaves) __attribute__((amdgpu_waves_per_eu(sr_unit_waves(LP, LA, LB))))
void sr3c_unit_kernel(const SRParams *__restrict__ prms, const SRWork *__restrict__ works,
                      long long *__restrict__ counts, const int w0, const int nwork) {
  constexpr int NCP = ncart(LP), NCA = ncart(LA), NCB = ncart(LB), NAB = NCA * NCB;
  constexpr int NBLK = NCP * NAB;
  constexpr int LAB = LA + LB, L = LAB + LP;
  constexpr int NH = nherm(L);
  constexpr int NT = sr_ntau(LP);
  constexpr bool WIDE = !sr_unit_class(LP, LA, LB);
  constexpr int NACC = WIDE ? NAB : NT * NAB;
  constexpr int RS = NH | 1;                    // odd: the units' sums start in distinct banks
  constexpr int NE = e_off(LB, LA, LB + 1);     // nonzero E coefficients per axis
  constexpr int NHAB = nherm(LAB);
  constexpr int kUnitCand = sr_unit_cand(LP, LA, LB), kUnitFill = sr_unit_fill(LP, LA, LB);
  constexpr int NBUF = kUnitCand * 32 > 64 * kUnitFl ? kUnitCand * 32 : 64 * kUnitFl;
  struct WaveLds {
    double buf[NBUF];  // candidate lists [entry][lane]; flush values [component][lane]
    double tc[kUnitTrip * kTripC];
    unsigned long long mx[kMaxCellsPerWave];
    float nf[kSRWinCap];
    int qii[kUnitQueue], qcw[kUnitQueue];  // pair image index; class | (largest window << kUnitClsBits)
    int rowcls[64], runcls[64], c2[64], rowend[64];
    unsigned cnt[3 * 64];  // per lane: terms, contractions, lattice vectors
    double u[uNum];        // the item's constants, read where they are used: in
    int n[nNum];           // registers they would push the lanes' sums to scratch
    double R[WIDE ? kWideUnits * RS : 1];         // wide classes: Hermite sums [unit][h]
    double E[WIDE ? kWideRows * 3 * NE : 1];      // and the E^ab of their images [row][axis]
  };
  __shared__ double2 s_boys[(L > 0 ? kBoysFineTab : 8 * kBoysFine) / 2];
  __shared__ WaveLds s_wave[kUnitWaves];

  {
    const double *tab = prms[0].boys_fine + (size_t)L * kBoysFineTab;
    double *dst = reinterpret_cast<double *>(s_boys);
    for (int i = threadIdx.x; i < (L > 0 ? kBoysFineTab : 8 * kBoysFine); i += 64 * kUnitWaves) dst[i] = tab[i];
  }
  __syncthreads();  // the only barrier of the workgroup
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wi = blockIdx.x * kUnitWaves + wv;
  if (wi >= nwork) return;
  WaveLds &sl = s_wave[wv];
  double *const s_buf = sl.buf, *const s_tc = sl.tc;
  float *const s_nf = sl.nf;
  int *const s_qii = sl.qii, *const s_qcw = sl.qcw;
  int *const s_rowcls = sl.rowcls, *const s_runcls = sl.runcls, *const s_c2 = sl.c2, *const s_rowend = sl.rowend;
  unsigned long long *const s_mx = sl.mx;
  unsigned *const s_cnt = sl.cnt;
  int *const s_cand = reinterpret_cast<int *>(s_buf);

  const SRWork wk = works[w0 + wi];
  const SRParams &prm = prms[wk.cell];
  const int S = wk.nslice;
  const Lattice &lat = prm.lat;
  const int nk = lat.nk;
  const double eps = prm.eps;
  double *const s_u = sl.u;
  int *const s_n = sl.n;
  for (int k = 0; k < 3; ++k) s_cnt[k * 64 + lane] = 0;
  {
    const Triplet tr = prm.trip[wk.trip];
    const Shell shP = prm.ax[tr.aux];
    const Pair pr = prm.pairs[tr.pair];
    const Shell shA = prm.ao[pr.sa];
    const Shell shB = prm.ao[pr.sb];
    const double omega = prm.omega, dR = prm.dR;
    const double fourpi_vol = 4.0 * kPi / lat.vol;
    const double pd = shA.a_d + shB.a_d;
    const double beta = shA.a_d * shB.a_d / pd;
    const double eta1 = sqrt(shP.a_d * pd / (shP.a_d + pd));
    const double eta2 = 1.0 / sqrt(1.0 / (eta1 * eta1) + 1.0 / (omega * omega));
    const double pref = tr.amp * fourpi_vol / (2.0 * beta);
    for (int w = lane; w < tr.nwin; w += 64) {
      const double R = w * dR;
      const double N = (R > prm.ncell_r0) ? fourpi_vol * 2.0 * (R + dR) * (R + dR) * dR : prm.ncell_nf;
      const double f = (R < 1e-12) ? 2.0 * (eta1 - eta2) * 0.564189583547756286948079451561 /* 1/sqrt(pi) */
                                   : (erf(eta1 * R) - erf(eta2 * R)) / R;
      s_nf[w] = (float)(pref * N * f);
    }
    const double xs = 1.0 / sqrt(2.0 * beta), inv2pi = 1.0 / (2.0 * kPi);
    s_u[uA] = shA.x, s_u[uA + 1] = shA.y, s_u[uA + 2] = shA.z;
    s_u[uB] = shB.x, s_u[uB + 1] = shB.y, s_u[uB + 2] = shB.z;
    s_u[uC] = shP.x, s_u[uC + 1] = shP.y, s_u[uC + 2] = shP.z;
    s_u[uBeta] = beta, s_u[uXstar] = xs, s_u[uGmax] = xs * exp(-0.5), s_u[uGrow] = pair_growth_c(beta);
    s_u[uR12min] = pr.R12min, s_u[uRc] = tr.rc_cut, s_u[uT1d] = shB.a_d / pd;
    const double *b = lat.b;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      for (int j = 0; j < 3; ++j) s_u[uRb + 3 * d + j] = b[3 * d + j] * inv2pi;
      s_u[uSp + d] = sqrt(b[3 * d] * b[3 * d] + b[3 * d + 1] * b[3 * d + 1] + b[3 * d + 2] * b[3 * d + 2]) * inv2pi;
      s_u[uOn + d] = 1.0 / lat.n[d];
      s_n[nMesh + d] = lat.n[d];
    }
    s_n[nPa] = shA.pptr, s_n[nPb] = shB.pptr, s_n[nPp] = shP.pptr;
    s_n[nTa] = shA.nprim, s_n[nTb] = shB.nprim, s_n[nTp] = shP.nprim;
    s_n[nFa] = shA.foff, s_n[nFb] = shB.foff, s_n[nFp] = shP.foff - prm.aux_f0, s_n[nDiag] = pr.diag;
    s_n[nNcb] = wk.ncb, s_n[nImg] = pr.img_off, s_n[nCoff] = pr.cls_off, s_n[nNsr] = pr.nsr_off, s_n[nW] = tr.nwin;
  }
  wave_sync();
  auto uni = [&](int i) -> int { return __builtin_amdgcn_readfirstlane(s_n[i]); };
  const int ntrip_p = uni(nTa) * uni(nTb) * uni(nTp);
  int tc0 = -1;  // first primitive triple of the chunk whose constants sit in LDS
  const bool logging = prm.logmag != nullptr;
  const double *a = lat.a;

  // lanes: rows of ncb cells, the lane's cell is fixed
  const int ncb = wk.ncb, rows = 64 / ncb;
  const int row = lane / ncb, gl = lane - row * ncb;
  const bool lane_on = row < rows;
  int i1x, i1y, i1z;
  {
    const int c1 = wk.cb0 + gl;
    i1x = c1 / (lat.n[1] * lat.n[2]), i1y = (c1 / lat.n[2]) % lat.n[1], i1z = c1 % lat.n[2];
  }
  const int nimg_all = __builtin_amdgcn_readfirstlane(prm.cls_off[uni(nCoff) + nk]);

  // wide classes: in the contraction the lanes are (part of the rows, cell, tau)
  const int nct = ncb * NT, nsub = WIDE ? 64 / nct : 1;
  const int sub2 = lane / nct, g2 = (lane - sub2 * nct) / NT, tau2 = lane - sub2 * nct - g2 * NT;
  int hix[WIDE ? (NHAB + 1) / 2 : 1];  // R index of Hermite order h + tau, two per register
  if constexpr (WIDE) {
    const int tx = tau_pow(LP, tau2, 0), ty = tau_pow(LP, tau2, 1), tz = tau_pow(LP, tau2, 2);
    static_for<0, (NHAB + 1) / 2>([&](auto I) {
      constexpr int h0 = 2 * decltype(I)::v, h1 = h0 + 1 < NHAB ? h0 + 1 : h0;
      constexpr int t0 = herm_pow(h0, 0), u0 = herm_pow(h0, 1), v0 = herm_pow(h0, 2);
      constexpr int t1 = herm_pow(h1, 0), u1 = herm_pow(h1, 1), v1 = herm_pow(h1, 2);
      hix[h0 / 2] = hidx(t0 + tx, u0 + ty, v0 + tz) | (hidx(t1 + tx, u1 + ty, v1 + tz) << 16);
    });
  }

  double acc[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i) acc[i] = 0.0;

  // geometry of pair image ii: B + n' - A
  auto image_vec = [&](int ii, double &bx, double &by, double &bz) {
    const double *nv = prm.img + 3 * ((size_t)s_n[nImg] + ii);
    bx = s_u[uB] + nv[0] - s_u[uA];
    by = s_u[uB + 1] + nv[1] - s_u[uA + 1];
    bz = s_u[uB + 2] + nv[2] - s_u[uA + 2];
  };

  // a window w is kept iff s_nf[w] >= thr (Eqs. S23-S24: R12 <= R12cut(w))
  auto window_thr = [&](double r12sq) -> double {
    const double R12 = sqrt(r12sq);
    double gx = (R12 <= s_u[uXstar]) ? s_u[uGmax] : R12 * exp(-s_u[uBeta] * r12sq);
    if constexpr (LAB > 0) {  // angular growth of the pair factor
      const double gr = fma(s_u[uGrow], R12, 1.0);
      double gp = gr;
#pragma unroll
      for (int i = 1; i < LAB; ++i) gp *= gr;
      gx *= gp;
    }
    return R12 <= s_u[uR12min] ? 0.0 : eps / gx;
  };

  int qh = 0, qn = 0, nxt = wk.slice;
  bool open = false;  // the accumulators hold images of the queue's first class
  for (;;) {
    // ---- refill: 64 images at a time, a lane tests one; the kept ones enter in list order
    while (qn < 64 && nxt < nimg_all) {
      const int ii = nxt + lane * S;
      int cls = 0, wm = -1;
      if (ii < nimg_all) {
        const int32_t *const coff = prm.cls_off + s_n[nCoff];
        int hi = nk - 1;
        while (cls < hi) {
          const int mid = (cls + hi + 1) >> 1;
          if (coff[mid] <= ii) cls = mid;
          else hi = mid - 1;
        }
        if (ii - coff[cls] < prm.nsr[s_n[nNsr] + cls] && !(prm.mask && !prm.mask[prm.cand_off[wk.trip] + ii])) {
          double bx, by, bz;
          image_vec(ii, bx, by, bz);
          const double thr = window_thr(bx * bx + by * by + bz * bz);
          wm = s_n[nW] - 1;
          while (wm >= 0 && !(s_nf[wm] >= thr)) --wm;
        }
      }
      const unsigned long long bal = __ballot(wm >= 0);
      if (wm >= 0) {
        const int at = (qh + qn + __popcll(bal & ((1ull << lane) - 1ull))) & (kUnitQueue - 1);
        s_qii[at] = ii;
        s_qcw[at] = cls | (wm << kUnitClsBits);
      }
      qn += __popcll(bal);
      nxt += 64 * S;
    }
    wave_sync();
    if (qn == 0) break;

    // ---- batch: whole runs of a class while they fit into the rows (or one
    // image in logging runs); a longer run goes in batches of its own, whose
    // sums stay in the registers until its last one.  Where the images hold more
    // lattice vectors than the lists, a batch is as few of them as fill the lists:
    // the rows are then shared out in proportion, and near and far images of a
    // run do not wait for one another.
    int m;
    bool ended;
    unsigned long long ends;
    {
      const bool in = lane < qn;
      const int cwj = in ? s_qcw[(qh + lane) & (kUnitQueue - 1)] : 0;
      const int cj = in ? (cwj & kUnitClsMask) : -1;
      const int cn = lane + 1 < qn ? (s_qcw[(qh + lane + 1) & (kUnitQueue - 1)] & kUnitClsMask)
                                   : (nxt >= nimg_all ? -2 : cj);
      // weight of the images up to this one; times vec, their lattice vectors per
      // cell (sphere volume)
      int cum = in ? sr_image_weight(cwj >> kUnitClsBits) : 0;
      const float vec = (float)(4.18879020478639098 * prm.dR * prm.dR * prm.dR / (lat.vol * nk));
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(cum, o, 64);
        cum += lane >= o ? up : 0;
      }
      const unsigned long long full = __ballot(in && (float)cum * vec >= (float)(rows * kUnitFill));
      // (the class after the queue's last image is known only once the list has ended)
      const int nibmax = logging ? 1 : min(min(rows, nxt >= nimg_all ? 64 : 63), full ? __ffsll((long long)full) : 64);
      const unsigned long long lim = nibmax >= 64 ? ~0ull : ((1ull << nibmax) - 1ull);
      ends = __ballot(in && (cj != cn || logging)) & lim;
      ended = ends != 0;
      // (the wide classes' accumulators are shared by the rows: one class at a time)
      m = !ended ? nibmax : (open || WIDE ? __ffsll((long long)ends) : 64 - __clzll((long long)ends));
      if (m < 64) ends &= (1ull << m) - 1ull;
      const bool lastj = in && ((ends >> lane) & 1ull);
      if (lastj) s_runcls[__popcll(ends & ((1ull << lane) - 1ull))] = cj;
      // rows per image in proportion to its lattice vectors, at least one each:
      // image j owns rows [s_rowend[j-1], s_rowend[j])
      const float inv_tot = 1.0f / (float)__shfl(cum, m - 1, 64);
      if (lane < m) s_rowend[lane] = sr_row_end(lane, m, rows, cum, inv_tot);
    }
    wave_sync();
    int slot = 0;
    {
      int hi = m - 1;
      while (slot < hi) {
        const int mid = (slot + hi) >> 1;
        if (s_rowend[mid] <= row) slot = mid + 1;
        else hi = mid;
      }
    }
    const int row0 = slot > 0 ? s_rowend[slot - 1] : 0;
    const int share = row - row0, lpu = s_rowend[slot] - row0;
    const bool act = lane_on;
    const int qa = (qh + slot) & (kUnitQueue - 1);
    const int ii_l = s_qii[qa], cw = s_qcw[qa];
    if (lane_on && gl == 0) s_rowcls[row] = cw & kUnitClsMask;
    double BAx, BAy, BAz;
    image_vec(ii_l, BAx, BAy, BAz);
    const double r12sq = BAx * BAx + BAy * BAy + BAz * BAz;
    const double thr = window_thr(r12sq);
    const double rmax = fmin(((cw >> kUnitClsBits) + 1) * prm.dR, s_u[uRc]);
    const double rmax2 = rmax * rmax;
    const double nm = 4.18879020478639098 * rmax2 * rmax / lat.vol + 1.0;
    // diffuse pair centre relative to the aux centre, and the box of lattice
    // coordinates M_d = i1_d + n_d j_d around it
    const double t1d = s_u[uT1d];
    const double X0x = s_u[uA] + t1d * BAx - s_u[uC], X0y = s_u[uA + 1] + t1d * BAy - s_u[uC + 1],
                 X0z = s_u[uA + 2] + t1d * BAz - s_u[uC + 2];
    int lo0, lo1, lo2, dim1, dim2, nbox;
    {
      const double *rb = s_u + uRb;
      const double f0 = -(rb[0] * X0x + rb[1] * X0y + rb[2] * X0z);
      const double f1 = -(rb[3] * X0x + rb[4] * X0y + rb[5] * X0z);
      const double f2 = -(rb[6] * X0x + rb[7] * X0y + rb[8] * X0z);
      const double sp0 = rmax * s_u[uSp], sp1 = rmax * s_u[uSp + 1], sp2 = rmax * s_u[uSp + 2];
      const double on0 = s_u[uOn], on1 = s_u[uOn + 1], on2 = s_u[uOn + 2];
      // (a box one too wide by rounding costs a test, not a term)
      lo0 = (int)ceil((f0 - sp0 - i1x) * on0 - 1e-9);
      lo1 = (int)ceil((f1 - sp1 - i1y) * on1 - 1e-9);
      lo2 = (int)ceil((f2 - sp2 - i1z) * on2 - 1e-9);
      const int dim0 = max(0, (int)floor((f0 + sp0 - i1x) * on0 + 1e-9) - lo0 + 1);
      dim1 = max(0, (int)floor((f1 + sp1 - i1y) * on1 + 1e-9) - lo1 + 1);
      dim2 = max(0, (int)floor((f2 + sp2 - i1z) * on2 + 1e-9) - lo2 + 1);
      // a mask, not a branch: lanes without a row run along with an empty box
      nbox = (dim0 * dim1 * dim2) & -(int)act;
    }
    const float inv12 = 1.0f / (float)max(dim1 * dim2, 1), inv2 = 1.0f / (float)max(dim2, 1);

    const double inv_dR = 1.0 / prm.dR;
    int q = share;
    for (;;) {
      // ---- the lane's next lattice vectors inside the screening windows
      int cnt = 0;
      while (q < nbox && cnt < kUnitCand) {
        int j0, j1, j2;
        sr_box_entry(q, dim1, dim2, inv12, inv2, j0, j1, j2);
        const int M0 = i1x + lat.n[0] * (lo0 + j0), M1 = i1y + lat.n[1] * (lo1 + j1),
                  M2 = i1z + lat.n[2] * (lo2 + j2);
        const double mx = X0x + M0 * a[0] + M1 * a[3] + M2 * a[6];
        const double my = X0y + M0 * a[1] + M1 * a[4] + M2 * a[7];
        const double mz = X0z + M0 * a[2] + M1 * a[5] + M2 * a[8];
        const double rc2 = mx * mx + my * my + mz * mz;
        if (rc2 <= rmax2) {
          const double rc = sqrt(rc2);
          const int w = (int)(rc * inv_dR);
          if ((rc <= s_u[uRc]) && (w < s_n[nW]) && (s_nf[w] >= thr)) {
            s_cand[cnt * 64 + lane] = pack3(M0, M1, M2);
            ++cnt;
          }
        }
        q += lpu;
      }
      s_cnt[2 * 64 + lane] += (unsigned)cnt;

      // ---- primitive triples: Hermite sums, then the contraction
      const int tt1 = __any(cnt > 0) ? ntrip_p : 0;
      for (int tt = 0; tt < tt1; ++tt) {
        if (tc0 < 0 || tt < tc0 || tt >= tc0 + kUnitTrip) {  // constants of the next chunk of triples
          wave_sync();
          tc0 = tt;
          const int t = tt + lane;
          if (lane < kUnitTrip && t < ntrip_p) {
            const int ntcp = s_n[nTp], ntb = s_n[nTb];
            const int kc = t % ntcp, kab = t / ntcp, kb = kab % ntb, ka = kab / ntb;
            const int ia = s_n[nPa] + ka, ib = s_n[nPb] + kb, ip = s_n[nPp] + kc;
            triple_consts<LP>(prm.ao_exp[ia], prm.ao_exp[ib], prm.ax_exp[ip], prm.ao_coef[ia], prm.ao_coef[ib],
                              prm.ax_coef[ip], prm.ao_c1s[ia], prm.ao_c1s[ib], prm.ax_c1s[ip], prm.omega, prm.acut,
                              s_tc + lane * kTripC);
          }
          wave_sync();
        }
        const double *const tcl = s_tc + (tt - tc0) * kTripC;
        const double Kab = exp(-tcl[2] * r12sq);
        // primitive screen: image-summed 1s estimate for this n' far below the target precision
        const int nt = (tcl[7] * Kab * nm < 1e-4 * eps) ? 0 : cnt;
        if (!__any(nt > 0)) continue;
        // offset of this primitive pair's centre from the aux centre at m = 0
        const double dt = tcl[1] - s_u[uT1d];
        const double dPx = X0x + dt * BAx, dPy = X0y + dt * BAy, dPz = X0z + dt * BAz;
        const double rho = tcl[3], th2 = tcl[4], th = tcl[5], m2rho = -2.0 * rho;
        double Rb[NH];
#pragma unroll
        for (int i = 0; i < NH; ++i) Rb[i] = 0.0;
        for (int e = 0; e < nt; ++e) {
          int M0, M1, M2;
          unpack3(s_cand[e * 64 + lane], M0, M1, M2);
          const double X = dPx + M0 * a[0] + M1 * a[3] + M2 * a[6];
          const double Y = dPy + M0 * a[1] + M1 * a[4] + M2 * a[7];
          const double Z = dPz + M0 * a[2] + M1 * a[5] + M2 * a[8];
          const double T = rho * (X * X + Y * Y + Z * Z);
          double g[L + 1];
          gvals_sr_fine<L>(T, th2, th, s_boys, g);
          double f = 1.0;
#pragma unroll
          for (int n = 1; n <= L; ++n) {
            f *= m2rho;
            g[n] *= f;
          }
          hermite_R_acc<L>(X, Y, Z, g, Rb);
        }
        wave_sync();  // (the constants below are read again, not kept over the loop)
        s_cnt[lane] += (unsigned)nt;
        if constexpr (!WIDE) s_cnt[64 + lane] += (unsigned)(nt > 0);
        if constexpr (WIDE) {
          // Where that leaves at least two rows fewer to contract, the lanes of a unit
          // are added up first (in a fixed order) and its first lane (share 0) contracts:
          // (d|dd) and (f|dd) of 8 atoms 2x2x2, omega 0.1, took 559 and 547 ms with a
          // contraction per lane and 12 vectors, 214 and 193 like this.
          const unsigned long long cells = (1ull << ncb) - 1ull;
          int has = nt > 0;
          const unsigned long long any = __ballot(has);
          const int act_rows = __popcll(__ballot(gl == 0 && lane_on && ((any >> (row * ncb)) & cells)));
          if (act_rows >= m + 2) {
            for (int o = 1; __any(lpu > o); o <<= 1) {
              const bool on = share + o < lpu;
              const int up = __shfl_down(has, o * ncb, 64);
              has |= on ? up : 0;
              static_for<0, NH>([&](auto I) {
                const double v = __shfl_down(Rb[decltype(I)::v], o * ncb, 64);
                Rb[decltype(I)::v] += on ? v : 0.0;
              });
            }
            has &= (int)(share == 0);
          }
          s_cnt[64 + lane] += (unsigned)has;
          // A few rows at a time: their lanes put the Hermite sums and E^ab (with
          // the prefactor in the x rows) into LDS, then lane (cell, tau) gathers
          // R[h + tau] of every row of its part and adds its NAB components.
          const unsigned long long bal = __ballot(has);
          const int RP = min(max(kWideUnits / ncb, 1), kWideRows);
          const double cK = tcl[6] * Kab, tb = tcl[1] - 1.0, oo2p = 0.5 * tcl[0], t1 = tcl[1];
          double sc = 1.0;  // (1/2g)^{(lP + |tau|)/2} of the lane's tau
#pragma unroll
          for (int i = 0; i < LP; ++i) sc *= (i < LP - 1 || tau2 < NCP) ? tcl[8] : 1.0;
          for (int r0 = 0; r0 < rows; r0 += RP) {
            if (!((bal >> (r0 * ncb)) & ((r0 + RP) * ncb >= 64 ? ~0ull : ((1ull << (RP * ncb)) - 1ull)))) continue;
            wave_sync();
            if (row >= r0 && row < r0 + RP && lane_on && ((bal >> (row * ncb)) & cells)) {
              double *Ru = sl.R + ((row - r0) * ncb + gl) * RS;
              static_for<0, NH>([&](auto I) { Ru[decltype(I)::v] = Rb[decltype(I)::v]; });
              if (gl == 0) {
                static_for<0, 3>([&](auto D) {
                  constexpr int d = decltype(D)::v;
                  const double ba = d == 0 ? BAx : (d == 1 ? BAy : BAz);
                  double E1[LA + 1][LB + 1][LAB + 1];
                  hermite_E<LA, LB>(t1 * ba, tb * ba, oo2p, E1);
                  double *Ed = sl.E + ((row - r0) * 3 + d) * NE;
                  static_for<0, (LA + 1) * (LB + 1)>([&](auto IJ) {
                    constexpr int i = decltype(IJ)::v / (LB + 1), j = decltype(IJ)::v % (LB + 1);
                    static_for<0, i + j + 1>([&](auto T) {
                      constexpr int tt_ = decltype(T)::v;
                      Ed[e_off(LB, i, j) + tt_] = d == 0 ? cK * E1[i][j][tt_] : E1[i][j][tt_];
                    });
                  });
                });
              }
            }
            wave_sync();
            for (int rr = sub2; rr < RP && r0 + rr < rows; rr += nsub) {
              if (sub2 >= nsub || !((bal >> ((r0 + rr) * ncb)) & cells)) continue;
              const double *Ru = sl.R + (rr * ncb + g2) * RS;
              const double *Ex = sl.E + rr * 3 * NE, *Ey = Ex + NE, *Ez = Ey + NE;
              double r[NHAB];
              static_for<0, NHAB>([&](auto I) {
                constexpr int h_ = decltype(I)::v;
                r[h_] = Ru[(h_ & 1) ? (hix[h_ / 2] >> 16) : (hix[h_ / 2] & 0xffff)];
              });
              static_for<0, NAB>([&](auto I) {
                constexpr int i = decltype(I)::v, ia = i / NCB, ib = i % NCB;
                constexpr int ax_ = crt_x(LA, ia), ay_ = crt_y(LA, ia), az_ = crt_z(LA, ia);
                constexpr int bx_ = crt_x(LB, ib), by_ = crt_y(LB, ib), bz_ = crt_z(LB, ib);
                double so = 0.0;
                static_for<0, ax_ + bx_ + 1>([&](auto T) {
                  constexpr int t_ = decltype(T)::v;
                  double st = 0.0;
                  static_for<0, ay_ + by_ + 1>([&](auto U) {
                    constexpr int u_ = decltype(U)::v;
                    double su = 0.0;
                    static_for<0, az_ + bz_ + 1>([&](auto V) {
                      constexpr int v_ = decltype(V)::v;
                      su += Ez[e_off(LB, az_, bz_) + v_] * r[hidx(t_, u_, v_)];
                    });
                    st += Ey[e_off(LB, ay_, by_) + u_] * su;
                  });
                  so += Ex[e_off(LB, ax_, bx_) + t_] * st;
                });
                acc[i] += sc * so;
              });
            }
          }
        } else {
        // E^ab per axis from P - A = t1 (B - A), P - B = (t1 - 1)(B - A)
        double Ex[LA + 1][LB + 1][LAB + 1], Ey[LA + 1][LB + 1][LAB + 1], Ez[LA + 1][LB + 1][LAB + 1];
        const double tb = tcl[1] - 1.0, oo2p = 0.5 * tcl[0];
        hermite_E<LA, LB>(tcl[1] * BAx, tb * BAx, oo2p, Ex);
        hermite_E<LA, LB>(tcl[1] * BAy, tb * BAy, oo2p, Ey);
        hermite_E<LA, LB>(tcl[1] * BAz, tb * BAz, oo2p, Ez);
        // factors (1/2g)^lP of |tau| = lP and (1/2g)^(lP - 1) of |tau| = lP - 2
        double cl = tcl[6] * Kab;
#pragma unroll
        for (int i = 1; i < LP; ++i) cl *= tcl[8];
        const double ct = LP > 0 ? cl * tcl[8] : cl;
        static_for<0, NT * NAB>([&](auto I) {
          constexpr int i = decltype(I)::v, tau = i / NAB, ia = (i % NAB) / NCB, ib = i % NCB;
          constexpr int tx = tau_pow(LP, tau, 0), ty = tau_pow(LP, tau, 1), tz = tau_pow(LP, tau, 2);
          constexpr int ax_ = crt_x(LA, ia), ay_ = crt_y(LA, ia), az_ = crt_z(LA, ia);
          constexpr int bx_ = crt_x(LB, ib), by_ = crt_y(LB, ib), bz_ = crt_z(LB, ib);
          double so = 0.0;
          static_for<0, ax_ + bx_ + 1>([&](auto T) {
            constexpr int t = decltype(T)::v;
            double st = 0.0;
            static_for<0, ay_ + by_ + 1>([&](auto U) {
              constexpr int u = decltype(U)::v;
              double su = 0.0;
              static_for<0, az_ + bz_ + 1>([&](auto V) {
                constexpr int v = decltype(V)::v;
                su += Ez[az_][bz_][v] * Rb[hidx(t + tx, u + ty, v + tz)];
              });
              st += Ey[ay_][by_][u] * su;
            });
            so += Ex[ax_][bx_][t] * st;
          });
          acc[i] += (tau < NCP ? ct : cl) * so;
        });
        }
      }
      if (!__any(q < nbox)) break;
    }

    // ---- end of the batch's last run: aux coefficients, sums over the rows of
    // each class, one store per element (every class of an item ends once)
    if (ended) {
      wave_sync();
      const int nrun = __popcll(ends);
      if (row < nrun) {
        const int cls = s_runcls[row], m0 = s_n[nMesh], m1 = s_n[nMesh + 1], m2 = s_n[nMesh + 2];
        // c2 = c1 + class (component-wise mod n)
        const int d0 = cls / (m1 * m2), d1 = (cls / m2) % m1, d2 = cls % m2;
        s_c2[lane] = (((i1x + d0) % m0) * m1 + (i1y + d1) % m1) * m2 + (i1z + d2) % m2;
      }
      if (logging && lane < kMaxCellsPerWave) s_mx[lane] = 0;
      constexpr int NF = NBLK < kUnitFl ? NBLK : kUnitFl;
      const int ncb_f = s_n[nNcb], nao = prm.nao;
      const size_t xplane = (size_t)prm.naux_b * nao * nao;
      double *const part = (wk.part >= 0) ? prm.part + wk.part : nullptr;
      wave_sync();
      // one element of the block of cell g, class target c2
      auto put = [&](int g, int c2, int comp, double v) {
        if (logging) {
          atomicMax(&s_mx[g], (unsigned long long)__double_as_longlong(fabs(v)));
          return;
        }
        if (v == 0.0) return;
        const int cc = wk.cb0 + g;
        if (part) {
          part[((size_t)g * nk + c2) * NBLK + comp] = v;
          return;
        }
        const int ic = comp / NAB, ia = (comp / NCB) % NCA, ib = comp % NCB;
        const size_t rowP = (size_t)(s_n[nFp] + ic) * nao;
        const int fa = s_n[nFa] + ia, fb = s_n[nFb] + ib;
        prm.X[(size_t)(cc * nk + c2) * xplane + (rowP + fa) * nao + fb] = v;
        if (!s_n[nDiag]) prm.X[(size_t)(c2 * nk + cc) * xplane + (rowP + fb) * nao + fa] = v;
      };
      if constexpr (WIDE) {
        constexpr int NFW = NAB < kUnitFl ? NAB : kUnitFl;
        static_for<0, (NAB + NFW - 1) / NFW>([&](auto F0) {
          constexpr int f0 = decltype(F0)::v * NFW;
          static_for<0, NFW>([&](auto J) {
            constexpr int j = decltype(J)::v;
            if constexpr (f0 + j < NAB) s_buf[j * 64 + lane] = acc[f0 + j];
          });
          wave_sync();
          for (int t = lane; t < ncb_f * NCP * NFW; t += 64) {
            const int g = t / (NCP * NFW), ic = (t / NFW) % NCP, j = t % NFW;
            if (f0 + j >= NAB) continue;
            double v = 0.0;
            for (int sb = 0; sb < nsub; ++sb) {
              const double *col = s_buf + j * 64 + sb * nct + g * NT;
              v += col[ic];
              for (int d = 0; d < 3; ++d) {
                const int c = tau_pow(LP, ic, d);
                if (LP >= 2 && c >= 2) v += (c == 3 ? 3.0 : 1.0) * col[NCP + tau_low(LP, ic, d)];
              }
            }
            put(g, s_c2[g], ic * NAB + f0 + j, v);
          }
          wave_sync();
        });
      } else
      static_for<0, (NBLK + NF - 1) / NF>([&](auto F0) {
        constexpr int f0 = decltype(F0)::v * NF;
        static_for<0, NF>([&](auto J) {
          constexpr int j = decltype(J)::v;
          if constexpr (f0 + j < NBLK) {
            constexpr int ic = (f0 + j) / NAB, ab = (f0 + j) % NAB;
            double v = acc[ic * NAB + ab];
            static_for<0, 3>([&](auto D) {
              constexpr int d = decltype(D)::v, c = tau_pow(LP, ic, d);
              if constexpr (c >= 2) v += (c == 3 ? 3.0 : 1.0) * acc[(NCP + tau_low(LP, ic, d)) * NAB + ab];
            });
            s_buf[j * 64 + lane] = v;
          }
        });
        wave_sync();
        for (int t = lane; t < nrun * ncb * NF; t += 64) {
          const int kg = t / NF, j = t - kg * NF, comp = f0 + j;
          if (comp >= NBLK) continue;
          const int k = kg / ncb_f, g = kg - k * ncb_f;
          const int cls = s_runcls[k];
          double v = 0.0;
          for (int r = 0; r < rows; ++r)
            if (s_rowcls[r] == cls) v += s_buf[j * 64 + r * ncb + g];
          put(g, s_c2[kg], comp, v);
        }
        wave_sync();
      });
      if (logging && lane < ncb)
        prm.logmag[(prm.cand_off[wk.trip] + s_qii[qh]) * nk + wk.cb0 + lane] = (float)__longlong_as_double((long long)s_mx[lane]);
#pragma unroll
      for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
      wave_sync();
    }
    open = !ended;
    qh = (qh + m) & (kUnitQueue - 1);
    qn -= m;
  }

  // ---- work counters (deterministic integer reduction), one slot per item
  long long cs[3] = {(long long)s_cnt[lane], (long long)s_cnt[64 + lane], (long long)s_cnt[2 * 64 + lane]};
#pragma unroll
  for (int k = 0; k < 3; ++k)
    for (int off = 32; off >= 1; off >>= 1) cs[k] += __shfl_xor(cs[k], off, 64);
  if (lane == 0) {
    long long *dst = counts + 4 * ((size_t)w0 + wi);
    dst[0] = cs[0];
    dst[1] = cs[1];
    dst[2] = cs[2];
    dst[3] = 0;
  }
}

// Sum the partial blocks of split work items (slice order) into X, direct and
// transposed entries.  One thread per element of a (work item, cell range).
__global__ void sr_reduce_kernel(const SRParams prm, const SRPartGroup *__restrict__ groups, int ngroups,
                                 int64_t nelem) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nelem) return;
  int lo = 0, hi = ngroups - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (groups[mid].elem_off <= gid) lo = mid;
    else hi = mid - 1;
  }
  const SRPartGroup g = groups[lo];
  const int64_t e = gid - g.elem_off;
  const Triplet tr = prm.trip[g.trip];
  const Pair pr = prm.pairs[tr.pair];
  const Shell shP = prm.ax[tr.aux], shA = prm.ao[pr.sa], shB = prm.ao[pr.sb];
  const int nca = ncart(shA.l), ncb = ncart(shB.l), nblk = ncart(shP.l) * nca * ncb;
  const int nk = prm.lat.nk;
  const int64_t blk = (int64_t)g.ncb * nk * nblk;
  double v = 0.0;
  for (int s = 0; s < g.nslice; ++s) v += prm.part[g.part + s * blk + e];
  const int comp = (int)(e % nblk);
  const int c2 = (int)((e / nblk) % nk);
  const int c1 = g.cb0 + (int)(e / ((int64_t)nblk * nk));
  const int ic = comp / (nca * ncb), ia = (comp / ncb) % nca, ib = comp % ncb;
  const size_t xplane = (size_t)prm.naux_b * prm.nao * prm.nao;
  const size_t rowP = (size_t)(shP.foff - prm.aux_f0 + ic) * prm.nao;
  prm.X[(size_t)(c1 * nk + c2) * xplane + (rowP + shA.foff + ia) * prm.nao + shB.foff + ib] += v;
  if (!pr.diag) prm.X[(size_t)(c2 * nk + c1) * xplane + (rowP + shB.foff + ib) * prm.nao + shA.foff + ia] += v;
}

hipError_t launch_sr_reduce(const SRParams &prm, const SRPartGroup *groups, int ngroups, int64_t nelem,
                            hipStream_t stream) {
  if (ngroups <= 0 || nelem <= 0) return hipSuccess;
  hipLaunchKernelGGL(sr_reduce_kernel, dim3((unsigned)((nelem + 255) / 256)), dim3(256), 0, stream, prm, groups,
                     ngroups, nelem);
  return hipGetLastError();
}

typedef void (*sr_kernel_t)(const SRParams *, const SRWork *, long long *, const int, const int);

#define RSGDF_SR_ENTRY(LP, LA, LB) &sr3c_unit_kernel<LP, LA, LB>
static const sr_kernel_t kSRTable[4][6] = {
    {RSGDF_SR_ENTRY(0, 0, 0), RSGDF_SR_ENTRY(0, 1, 0), RSGDF_SR_ENTRY(0, 1, 1), RSGDF_SR_ENTRY(0, 2, 0),
     RSGDF_SR_ENTRY(0, 2, 1), RSGDF_SR_ENTRY(0, 2, 2)},
    {RSGDF_SR_ENTRY(1, 0, 0), RSGDF_SR_ENTRY(1, 1, 0), RSGDF_SR_ENTRY(1, 1, 1), RSGDF_SR_ENTRY(1, 2, 0),
     RSGDF_SR_ENTRY(1, 2, 1), RSGDF_SR_ENTRY(1, 2, 2)},
    {RSGDF_SR_ENTRY(2, 0, 0), RSGDF_SR_ENTRY(2, 1, 0), RSGDF_SR_ENTRY(2, 1, 1), RSGDF_SR_ENTRY(2, 2, 0),
     RSGDF_SR_ENTRY(2, 2, 1), RSGDF_SR_ENTRY(2, 2, 2)},
    {RSGDF_SR_ENTRY(3, 0, 0), RSGDF_SR_ENTRY(3, 1, 0), RSGDF_SR_ENTRY(3, 1, 1), RSGDF_SR_ENTRY(3, 2, 0),
     RSGDF_SR_ENTRY(3, 2, 1), RSGDF_SR_ENTRY(3, 2, 2)},
};

// pair class index of (la, lb) with la >= lb
hipError_t launch_sr3c(int lP, int pc, const SRParams *prms, const SRWork *works, long long *counts, int w0,
                       int nwork, hipStream_t stream) {
  if (nwork <= 0) return hipSuccess;
  hipLaunchKernelGGL(kSRTable[lP][pc], dim3((unsigned)((nwork + kUnitWaves - 1) / kUnitWaves)), dim3(64 * kUnitWaves), 0,
                     stream, prms, works, counts, w0, nwork);
  return hipGetLastError();
}

}  // namespace rsgdf

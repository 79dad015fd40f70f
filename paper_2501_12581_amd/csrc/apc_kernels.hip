// HIP kernels (gfx950) for the APC hot path.
//
// One frame = for the listed subdomains:
//   k_bin        boundary faces of each subdomain -> (tile, subdomain) bins
//                (count pass, exclusive scan, fill pass)
//   k_moments    one 64-lane wavefront per 8x8 pixel tile: per subdomain,
//                collect the boundary faces where each pixel ray enters the
//                subdomain, walk the ray tet by tet from each entry to where
//                it leaves the subdomain, queue the chords, cut them at the
//                global sampling lattice and add a*z^j per piece (Alg. 2)
//                (with every subdomain on one GPU it also sums them: the
//                global image; else per-subdomain images, dense or as tiles
//                of the (tile, subdomain) pairs that have boundary faces)
//   k_sum_moments / k_sum_tiles  canonical-order FP64 sum of per-subdomain
//                images or tiles (the paper's moment Allreduce, Section 4.1)
//   k_resolve    stage two, plain form: per tile a walker wavefront walks the
//                rays again and hands each chord's end (depth, scalar) through
//                LDS to an evaluator wavefront, which cuts it into the pieces
//                stage one had, forms their optical and warped depths, evaluates the
//                moment bound of its pixel (Alg. 3) and weights the piece's
//                colour by T = exp(-b0 F) (Alg. 1 second loop, Section 4.2)
//   k_eval       the same evaluation over pieces stage one kept (variant)
//   k_sum_images canonical-order sum of partial images + renormalisation
//
// Geometry.  A ray crosses a face iff its Plücker side products with the
// face's three edges share one sign.  Every edge product is computed with one
// formula whose two orientations give exactly opposite values, and an exact
// zero counts as positive in the orientation from the lower vertex id to the
// higher; the entry test of one subdomain and the exit test of the walk in
// its neighbour therefore see identical signs for the face they share, so
// every ray crosses each subdomain interface exactly once (no gaps, no double
// counting).  The barycentric coordinates of the crossing point are the three
// edge products of the face, which give the depth t and the scalar there.  Functions whose results must agree
// bit for bit between the two passes or between the entry test and the walk
// are compiled without floating-point contraction.
#include <float.h>

// Products and sums are fused within an expression only, as written: fused across statements too (the compiler's
// default) it depends on the code around, and the variants of a kernel (tiles from a grid or a queue, by pair)
// would round differently.
#pragma clang fp contract(on)

#include "apc_cut.h"
#include "apc_internal.h"
#include "apc_mboit.h"

namespace apc {
namespace {

constexpr int WAVE = 64;
constexpr int E_MAX = 8;     // entries per ray held at once (more are handled in further rounds)
constexpr int CHUNK = 32;    // boundary faces staged in LDS at a time

// Outward vertex order of the face opposite vertex f of a positively oriented tet: the local vertices f ^ 1,
// f ^ 2, f ^ 3 in this order; inward: f ^ 1, f ^ 3, f ^ 2.

__device__ __forceinline__ int sel4(const int4& v, int i) {
  return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}
// b where m is all ones, a where it is 0 (v_bfi_b32: no compare, and nothing for the compiler to branch on)
__device__ __forceinline__ int bit_select(int m, int a, int b) { return (m & b) | (~m & a); }
__device__ __forceinline__ unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool lane_of(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// The block's number in a launch over wide_grid.
__device__ __forceinline__ int64_t flat_block() { return int64_t(blockIdx.y) * gridDim.x + blockIdx.x; }

// Blocks are dispatched round-robin over the 8 XCDs (block b runs on XCD
// b % 8).  The tiles are handed out in runs of XCD_RUN consecutive tiles, so
// neighbouring tiles (which read the same tets) share one XCD's L2, and
// every XCD gets runs from all over the image: the work of a view is
// concentrated where the volume projects, and one contiguous band of the
// image per XCD gave the busiest XCD twice the mean work.  Round k of 8 runs
// (runs 8k .. 8k+7) goes to the XCDs rotated by k: with run c on XCD c % 8,
// an image row of 4 runs (2048 pixels of 8-wide tiles) put the same quarter
// of every row on one XCD.  The blocks beyond the last whole round take the
// remaining tiles in bands.
#ifndef APC_XCD_RUN
#define APC_XCD_RUN 64
#endif
constexpr int XCD_RUN = APC_XCD_RUN;
__device__ __forceinline__ int xcd_tile(int b, int nb, int run = XCD_RUN) {
  const int whole = nb / (8 * run) * (8 * run);
  if (b < whole) {
    const int x = b & 7, i = b >> 3;
    const int k = i / run;
    return (k * 8 + ((x + k) & 7)) * run + (i - k * run);
  }
  b -= whole;
  nb -= whole;
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, i = b >> 3;
  return whole + x * q + (x < r ? x : r) + i;
}

// Persistent launches (a work queue): as many workgroups as the device holds
// at once, each taking tile after tile until none is left.  The tiles are
// the ones the ordinary launch of nb workgroups would give, per XCD in the
// same order: XCD x owns the tiles of the workgroups b = 8k + x, handed out
// by its own counter q[x]; a workgroup whose XCD has none left takes the next
// one of the following XCDs.  Called by one lane; -1 when all are taken.
__device__ __forceinline__ int queue_take(int* q, int nb) {
  const int x = blockIdx.x & 7;
  for (int d = 0; d < 8; ++d) {
    const int y = (x + d) & 7;
    const int own = (nb - y + 7) >> 3;  // workgroups b < nb with b % 8 == y
    if (__hip_atomic_load(q + y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= own) continue;
    const int k = atomicAdd(q + y, 1);
    if (k < own) return xcd_tile(8 * k + y, nb);
  }
  return -1;
}

// A pixel ray in FP64, as what the walk needs of it: with o the origin (moved forward by t_mid), d the unit
// direction and (a, b, d) a right-handed orthonormal frame, the vectors d, a, b and the offsets -d.o, -a.o, -b.o
// (a point's coordinates in the frame are then three fused multiply-adds each; the offsets round to ~1e-16 of
// the distance to the origin, far below the FP32 rounding of the vertex positions themselves).
struct Ray {
  double dx, dy, dz, ax, ay, az, bx, by, bz, od, oa, ob;
};

__device__ __forceinline__ Ray pixel_ray(const FrameDev& f, int i, int j) {
#pragma clang fp contract(off)
  const double a = double(j) + 0.5, b = double(i) + 0.5;
  Ray r;
  double dx, dy, dz, ox, oy, oz;
  if (f.proj == 0) {
    ox = f.ceye[0] + a * f.cright[0] + b * f.cdown[0];
    oy = f.ceye[1] + a * f.cright[1] + b * f.cdown[1];
    oz = f.ceye[2] + a * f.cright[2] + b * f.cdown[2];
    dx = f.cdir[0];
    dy = f.cdir[1];
    dz = f.cdir[2];
  } else {
    ox = f.ceye[0];
    oy = f.ceye[1];
    oz = f.ceye[2];
    const double aa = a - 0.5 * double(f.W), bb = b - 0.5 * double(f.H);
    dx = f.cdir[0] + aa * f.cright[0] + bb * f.cdown[0];
    dy = f.cdir[1] + aa * f.cright[1] + bb * f.cdown[1];
    dz = f.cdir[2] + aa * f.cright[2] + bb * f.cdown[2];
  }
  const double inv = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
  r.dx = dx * inv;
  r.dy = dy * inv;
  r.dz = dz * inv;
  {
    // a = d x h / |d x h| for a coordinate axis h far from parallel to d
    const bool xs = fabs(r.dx) < 0.9;
    const double hx = xs ? 1.0 : 0.0, hy = xs ? 0.0 : 1.0;
    const double ax = -r.dz * hy, ay = r.dz * hx, az = r.dx * hy - r.dy * hx;
    const double ia = 1.0 / sqrt(ax * ax + ay * ay + az * az);
    r.ax = ax * ia;
    r.ay = ay * ia;
    r.az = az * ia;
    r.bx = r.dy * r.az - r.dz * r.ay;
    r.by = r.dz * r.ax - r.dx * r.az;
    r.bz = r.dx * r.ay - r.dy * r.ax;
  }
  // depth 0 at the middle of the depth range
  ox = ox + f.t_mid * r.dx;
  oy = oy + f.t_mid * r.dy;
  oz = oz + f.t_mid * r.dz;
  r.od = -(r.dx * ox + r.dy * oy + r.dz * oz);
  r.oa = -(r.ax * ox + r.ay * oy + r.az * oz);
  r.ob = -(r.bx * ox + r.by * oy + r.bz * oz);
  return r;
}

// A vertex as seen from one ray: scalar, depth t = d.(P-o) (FP64) and its
// coordinates u = a.(P-o), v = b.(P-o) in the plane perpendicular to the ray,
// computed in FP64 and rounded to FP32 (near the ray |u|, |v| are about a
// cell's size, so the rounding is ~1e-7 of a cell, not of the distance to
// the eye).
struct VS {
  float s, u, v;
  double t;
};

__device__ __forceinline__ VS vstate(const Ray& r, float4 p) {
  const double x = p.x, y = p.y, z = p.z;
  VS v;
  v.s = p.w;
  v.t = fma(r.dx, x, fma(r.dy, y, fma(r.dz, z, r.od)));
  v.u = float(fma(r.ax, x, fma(r.ay, y, fma(r.az, z, r.oa))));
  v.v = float(fma(r.bx, x, fma(r.by, y, fma(r.bz, z, r.ob))));
  return v;
}

// Oriented Plücker side product d.((a-o) x (b-o)) of the ray with the edge
// a -> b: only the components perpendicular to d contribute, so it is the 2D
// cross product u_a v_b - v_a u_b.  Without contraction the two orientations
// of an edge give exactly opposite values (the products are the same two
// roundings in either order), so every test that meets the edge sees one
// value up to sign; an exact zero counts as positive in the orientation from
// the lower vertex id to the higher (the callers' part: zeros are rare).
__device__ __forceinline__ float side(const VS& a, const VS& b) {
#pragma clang fp contract(off)
  return a.u * b.v - a.v * b.u;
}
__device__ __forceinline__ float zero_side(bool low_to_high) { return low_to_high ? FLT_MIN : -FLT_MIN; }

// Crossing point of the ray with the face (A, B, C) whose oriented products
// pAB, pBC, pCA are all positive: barycentric weights (pBC, pCA, pAB).  The
// depth is A's FP64 depth plus the weighted depth differences across the face
// (at most a cell's extent, so FP32 keeps them to ~1e-7 of a cell, the
// precision of the weights themselves); the scalar likewise.
__device__ __forceinline__ void face_point(const VS& A, const VS& B, const VS& C, float pAB, float pBC, float pCA,
                                           double& t, float& s) {
  const float inv = __builtin_amdgcn_rcpf(fmaxf(pBC + pCA + pAB, FLT_MIN));  // 1 ulp; both passes alike
  t = A.t + double(fmaf(pCA, float(B.t - A.t), pAB * float(C.t - A.t)) * inv);
  s = fmaf(fmaf(pCA, B.s - A.s, pAB * (C.s - A.s)), inv, A.s);
}

// a or b, field by field (value selects: no store through a selected address)
__device__ __forceinline__ VS pick(bool c, const VS& a, const VS& b) {
  VS r;
  r.s = c ? a.s : b.s;
  r.u = c ? a.u : b.u;
  r.v = c ? a.v : b.v;
  r.t = c ? a.t : b.t;
  return r;
}

// face_point with the vertex `base` (0 A, 1 B, 2 C) first: the one with the
// smallest id, so a walk that leaves its subdomain (or the mesh) through a
// face and the entry test of the tet behind it (which list the face's vertices
// in different rotations) get the same depth bit for bit.
__device__ __forceinline__ void face_point_from(int base, const VS& A, const VS& B, const VS& C, float pAB, float pBC,
                                                float pCA, double& t, float& s) {
  const bool b1 = base == 1, b2 = base == 2;
  face_point(pick(b1, B, pick(b2, C, A)), pick(b1, C, pick(b2, A, B)), pick(b1, A, pick(b2, B, C)),
             b1 ? pBC : (b2 ? pCA : pAB), b1 ? pCA : (b2 ? pAB : pBC), b1 ? pAB : (b2 ? pBC : pCA), t, s);
}

// A boundary face staged in LDS, vertices in outward order of its tet.
struct FaceL {
  int code;  // (tet << 2) | face
  int id0, id1, id2;
  float4 p0, p1, p2;
};

// Which of the face's vertices 0, 1, 2 (outward order) in the slots A, B, C =
// vertices 0, 2, 1 (inward order) has the smallest id.
__device__ __forceinline__ int first_slot(int id0, int id1, int id2) {
  return id0 < id1 && id0 < id2 ? 0 : (id2 < id1 ? 1 : 2);
}

// Does the ray enter the face's tet through it (vertices in outward order)?
// On success also the entry depth.
__device__ __forceinline__ bool enters(const Ray& r, int id0, int id1, int id2, float4 p0, float4 p1, float4 p2,
                                       double& t) {
  const VS a = vstate(r, p0), b = vstate(r, p1), c = vstate(r, p2);
  float sab = side(a, b), sbc = side(b, c), sca = side(c, a);
  if (sab == 0.0f) sab = zero_side(id0 < id1);
  if (sbc == 0.0f) sbc = zero_side(id1 < id2);
  if (sca == 0.0f) sca = zero_side(id2 < id0);
  if (!(sab < 0.0f && sbc < 0.0f && sca < 0.0f)) return false;
  // inward order (a, c, b): pi(a->c) = -sca, pi(c->b) = -sbc, pi(b->a) = -sab
  float s;
  face_point_from(first_slot(id0, id1, id2), a, c, b, -sca, -sbc, -sab, t, s);
  return true;
}

// Per-lane event counts, summed over the wavefront at the end of a kernel.  Events that are rare by design
// (a walk cut off by its step limit, an exit face chosen by the tie fallback, an entry list or buffer that
// overflowed) go straight to the device counters instead, so they hold no register in the walk.
struct LaneCount {
  unsigned pieces, entries, nonpd, segments;
  unsigned w_pieces, w_steps, w_tabled, w_fallback;  // counted for the whole wavefront at once
  unsigned long long* ctr;
  __device__ void rare(int which, unsigned n = 1u) {
    if (n) atomicAdd(ctr + which, (unsigned long long)n);
  }
};

// Transfer-function table coordinate of scalar s, clamped to the table: entry
// i0 in [0, n_tf - 1] and fraction fr (0 at the last entry).
__device__ __forceinline__ void tf_coord(const FrameDev& f, float s, int& i0, float& fr) {
  const float u = __builtin_amdgcn_fmed3f((s - f.s_min) * f.tf_scale, 0.0f, float(f.n_tf - 1));
  i0 = int(u);
  fr = __builtin_amdgcn_fractf(u);
}

// Kappa times a table entry's alpha, within what the differences of two and their products with a fraction can
// hold: an infinite product caps every piece all the same, and infinity times no alpha is none.
__device__ __forceinline__ float kappa_alpha(const FrameDev& f, float alpha) {
  const float k = f.kappa * alpha;
  return k == k ? __builtin_amdgcn_fmed3f(k, -0.25f * FLT_MAX, 0.25f * FLT_MAX) : 0.0f;
}

// Optical depth of a piece (Alg. 2: absorbance capped) from kappa times the
// transfer function's alpha at its scalar and its length, and its warped depth
// (log depth rescaled to [-1, 1], clamped to the range) from its mid depth
// measured from the eye over the geometric mean of the range's ends: the
// logarithm is 0 in the middle of the range, so the hardware's relative error
// (about an ulp, mostly of one sign) is one of z, with no larger number
// subtracted from it.
__device__ __forceinline__ float piece_a(const FrameDev& f, float kA, float len) {
  return __builtin_amdgcn_fmed3f(kA * len, 0.0f, f.amax);  // min with the cap (the product is >= 0)
}
__device__ __forceinline__ double piece_z(const FrameDev& f, float wt) {
  return double(__builtin_amdgcn_fmed3f(__builtin_amdgcn_logf(wt), -f.lg_half, f.lg_half)) * f.z_scale;
}

// Opacity 1 - e^-a of a piece of optical depth a >= 0: below 0.35 the Taylor
// polynomial of degree 7 (the first omitted term is under 2e-8 of the value),
// above it the hardware exponential (no cancellation there: e^-a < 0.71).
__device__ __forceinline__ float opacity(float a) {
  float p = 1.0f / 5040.0f;
  p = fmaf(p, -a, 1.0f / 720.0f);
  p = fmaf(p, -a, 1.0f / 120.0f);
  p = fmaf(p, -a, 1.0f / 24.0f);
  p = fmaf(p, -a, 1.0f / 6.0f);
  p = fmaf(p, -a, 0.5f);
  p = fmaf(p, -a, 1.0f);
  return a < 0.35f ? a * p : 1.0f - __expf(-a);
}

// Where a walk stands: the face (A, B, C) through which the ray entered the
// current tet, with its positive side products; the code (tet << 2) | f of
// that tet and the local index f of the vertex opposite the face; and how the
// face's vertices A, B, C sit in the tet: slot i (A 0, B 1, C 2) holds the
// vertex at position (i + rot) mod 3 of the inward order f ^ 1, f ^ 3, f ^ 2.
struct WalkPos {
  VS A, B, C;
  float pAB, pBC, pCA;
  int code;
  int rot;
};

// The walk record of a tet entered through its face f, 32 bytes: the vertex
// opposite f, the codes of the tets behind the three other faces (in the
// order of their opposite vertices' positions; -1 where that face lies on the
// mesh hull or leads out of the subdomain) and packed bits about them
// (k_walk_records).  All a step needs, in two loads that go out together.
struct WalkRec {
  float4 v;
  int4 n;
};
__device__ __forceinline__ WalkRec walk_rec(const MeshDev& M, int code) {
  const int4* p = M.wrec + 2 * size_t(unsigned(code));
  WalkRec r;
  r.v = *reinterpret_cast<const float4*>(p);
  r.n = p[1];
  return r;
}

// One step of the walk through the tet of record `rec`: the depth and scalar
// where the ray leaves it (tout >= tin); the position moves to the tet behind
// (w.code < 0 when the exit face lies on the mesh hull or leads out of the
// subdomain).  Returns whether the chord has any length.  The whole wavefront
// takes the step: a lane that walks no more computes with a record it does not
// use, and its code stays -1 (with the step under a condition the compiler
// copies the whole position around it).  No vertex ids are needed: what they
// decide (the sign of a zero product, the first vertex of a face that leaves
// the subdomain, how the next tet numbers the face's vertices) is in the
// record's bits.
__device__ __forceinline__ bool walk_step(const Ray& r, WalkPos& w, const WalkRec& rec, double tin, double& tout,
                                          float& sout, LaneCount& cnt) {
  const VS D = vstate(r, rec.v);
  const unsigned info = unsigned(rec.n.w);
  float qA = side(D, w.A), qB = side(D, w.B), qC = side(D, w.C);
  const bool alive = w.code >= 0;
  if ((fminf(fminf(fabsf(qA), fabsf(qB)), fabsf(qC)) == 0.0f) & alive) {
    const int p1 = w.rot >= 2 ? w.rot - 2 : w.rot + 1, p2 = w.rot >= 1 ? w.rot - 1 : 2;
    if (qA == 0.0f) qA = zero_side((info >> (12 + w.rot)) & 1);
    if (qB == 0.0f) qB = zero_side((info >> (12 + p1)) & 1);
    if (qC == 0.0f) qC = zero_side((info >> (12 + p2)) & 1);
  }
  // exit through the face opposite X where q(next of X) > 0 > q(previous of X)
  const unsigned long long a = ballot(qA > 0.0f), b = ballot(qB > 0.0f), c = ballot(qC > 0.0f);
  bool x0 = lane_of(b & ~c), x1 = lane_of(c & ~a), x2 = lane_of(a & ~b);
  const bool none = alive & lane_of((a & b & c) | ~(a | b | c));
  if (none) {  // sign pattern no line can have (rounding near a vertex): least-violated face
    const float m0 = fminf(qB, -qC), m1 = fminf(qC, -qA), m2 = fminf(qA, -qB);
    x0 = m0 >= m1 && m0 >= m2;
    x1 = !x0 && m1 >= m2;
    x2 = !x0 && !x1;
    cnt.rare(C_FALLBACK);
  }
  // The exit face replaces X by D in place: (D, B, C), (A, D, C) and
  // (A, B, D) are rotations of the exit faces (B, C, D), (C, A, D) and
  // (A, B, D), so the cyclic order with positive products is kept.
  w.pAB = x0 ? qB : (x1 ? -qA : w.pAB);
  w.pBC = x1 ? qC : (x2 ? -qB : w.pBC);
  w.pCA = x2 ? qA : (x0 ? -qC : w.pCA);
  if (none) {  // weights never negative
    w.pAB = fmaxf(w.pAB, 0.0f);
    w.pBC = fmaxf(w.pBC, 0.0f);
    w.pCA = fmaxf(w.pCA, 0.0f);
    asm volatile("; rare: kept a branch");
  }
  w.A = pick(x0, D, w.A);
  w.B = pick(x1, D, w.B);
  w.C = pick(x2, D, w.C);
  const int x = x1 ? 1 : (x2 ? 2 : 0);
  unsigned y = unsigned(x + w.rot);  // position of X: its face's place in the record
  y = min(y, y - 3u);
  // the face's place in the record is 0, 1 or 2: bit 0 and bit 1 of y select
  const int nb = bit_select(__builtin_amdgcn_sbfe(int(y), 1, 1),
                            bit_select(__builtin_amdgcn_sbfe(int(y), 0, 1), rec.n.x, rec.n.y), rec.n.z);
  face_point(w.A, w.B, w.C, w.pAB, w.pBC, w.pCA, tout, sout);
  if (alive & (nb < 0)) {  // leaves the subdomain
    unsigned base = unsigned(x) + ((info >> (6 + 2 * y)) & 3u);
    base = min(base, base - 3u);
    face_point_from(int(base), w.A, w.B, w.C, w.pAB, w.pBC, w.pCA, tout, sout);
  }
  unsigned rot = unsigned(w.rot) + ((info >> (2 * y)) & 3u);
  w.rot = int(min(rot, rot - 3u));
  w.code = alive ? nb : -1;
  const bool forward = alive & (tout > tin);
  tout = forward ? tout : tin;
  return forward;
}

// A queue of chords per lane in LDS (lane-minor: the 64 lanes hit distinct
// banks): where each ends, depth and scalar.
template <int SLOTS>
struct ChordRing {
  static_assert((SLOTS & (SLOTS - 1)) == 0, "the ring size is a power of two");
  double t[SLOTS * WAVE];
  float s[SLOTS * WAVE];
};
constexpr int CHORDS = 8;  // stage one's queue

// Per-lane list of entries (depth, face code) in LDS, kept sorted by
// (depth, code); lane-minor layout so the 64 lanes hit distinct banks.
struct EntryList {
  float* t;  // [E_MAX][WAVE]
  int* c;
  int lane;
  __device__ float& T(int e) { return t[e * WAVE + lane]; }
  __device__ int& Cd(int e) { return c[e * WAVE + lane]; }
};

__device__ __forceinline__ bool key_less(float ta, int ca, float tb, int cb) {
  return ta < tb || (ta == tb && ca < cb);
}

// Stage a chunk of boundary-face records of one bin into LDS.
__device__ __forceinline__ void stage_faces(const MeshDev& M, const int* rec, int n, FaceL* faces, int lane) {
  if (lane < n) {
    int code = rec[lane];
    int t = code >> 2, fc = code & 3;
    int4 tv = M.tet[2 * t];
    FaceL F;
    F.code = code;
    F.id0 = sel4(tv, fc ^ 1);
    F.id1 = sel4(tv, fc ^ 2);
    F.id2 = sel4(tv, fc ^ 3);
    F.p0 = M.vert[F.id0];
    F.p1 = M.vert[F.id1];
    F.p2 = M.vert[F.id2];
    faces[lane] = F;
  }
}

// LDS writes of a wavefront visible to all its lanes (no workgroup barrier)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The next (up to EMAX) entries of this lane's ray into one subdomain after
// the key (last_t, last_c), sorted by (depth, code) into L; returns how many,
// and sets `more` when there were others beyond them.  Must be called by the
// whole wavefront (it stages faces cooperatively into the wavefront's own LDS
// slice, so a workgroup may hold several wavefronts walking different tiles).
template <int EMAX>
__device__ int collect_entries(const MeshDev& M, const Ray& r, bool want, const int* rec, int n_rec, FaceL* faces,
                               EntryList& L, float last_t, int last_c, bool& more) {
  int n = 0;
  more = false;
  for (int c0 = 0; c0 < n_rec; c0 += CHUNK) {
    int nc = min(CHUNK, n_rec - c0);
    wave_sync();  // every lane is done with the previous chunk
    stage_faces(M, rec + c0, nc, faces, L.lane);
    wave_sync();
    if (!want) continue;
    for (int k = 0; k < nc; ++k) {
      const FaceL& F = faces[k];
      double t;
      if (!enters(r, F.id0, F.id1, F.id2, F.p0, F.p1, F.p2, t)) continue;
      const float et = float(t);  // sort key: the entry depth rounded to FP32
      if (!key_less(last_t, last_c, et, F.code)) continue;  // walked in an earlier round
      if (n == EMAX) {
        more = true;
        if (!key_less(et, F.code, L.T(n - 1), L.Cd(n - 1))) continue;
        --n;  // evict the largest
      }
      int pos = n;
      while (pos > 0 && key_less(et, F.code, L.T(pos - 1), L.Cd(pos - 1))) {
        L.T(pos) = L.T(pos - 1);
        L.Cd(pos) = L.Cd(pos - 1);
        --pos;
      }
      L.T(pos) = et;
      L.Cd(pos) = F.code;
      ++n;
    }
  }
  return n;
}

// Starts a walk at an entry of the list, `code` = (tet << 2) | face: the state
// at the boundary face (the ray enters there: it was listed so) and the entry
// depth and scalar, the ones the entry test found.
__device__ __forceinline__ void start_walk(const MeshDev& M, const Ray& r, int code, WalkPos& w, double& t, float& s) {
  const int fc = code & 3;
  const int4 tv = M.tet[2 * (code >> 2)];
  const int i0 = sel4(tv, fc ^ 1), i1 = sel4(tv, fc ^ 2), i2 = sel4(tv, fc ^ 3);
  w.A = vstate(r, M.vert[i0]);
  w.C = vstate(r, M.vert[i1]);
  w.B = vstate(r, M.vert[i2]);
  w.pAB = side(w.A, w.B);
  w.pBC = side(w.B, w.C);
  w.pCA = side(w.C, w.A);
  w.pAB = w.pAB == 0.0f ? FLT_MIN : w.pAB;
  w.pBC = w.pBC == 0.0f ? FLT_MIN : w.pBC;
  w.pCA = w.pCA == 0.0f ? FLT_MIN : w.pCA;
  w.code = code;
  w.rot = 0;
  face_point_from(first_slot(i0, i1, i2), w.A, w.B, w.C, w.pAB, w.pBC, w.pCA, t, s);
}

// All entries of this lane's ray into one subdomain, walked in (depth, code)
// order.  Handles more than E_MAX entries by repeated rounds that pick the
// next E_MAX entries after the last one walked.  Must be called by the whole
// wavefront.
//
// A walk step hands its chord to the lane's queue, and the pieces are cut and
// summed in rounds of one piece per lane that run only while most lanes have
// one (ROUND_LANES of 64): a tet's chord holds 1 to 6 pieces, and a loop over
// one chord's pieces ran as long as the lane with the most, at 62 % of the
// lanes on average.  The record of the next tet is asked for before the
// rounds and used after them.  Bound by vector instructions issued (FP64
// among them at the same rate).  Measured, m = 8, 2560^2 on 12.6M tets: 17.4 ms
// with a loop per chord and 64-byte records, 12.2 ms now (56 lanes
// the same); 1024^2 on 1.6M tets 1.72 -> 1.18 ms at m = 6.
constexpr int ROUND_LANES = 48;
template <class Sink>
__device__ void walk_subdomain(const MeshDev& M, const FrameDev& f, const Ray& r, bool valid, const int* rec,
                               int n_rec, FaceL* faces, EntryList& L, ChordRing<CHORDS>& ring, Sink& sink,
                               LaneCount& cnt) {
  float last_t = -FLT_MAX;
  int last_c = -1;
  bool more = true;
  while (true) {
    bool want = valid && more;
    if (!__any(want)) break;
    const int n = collect_entries<E_MAX>(M, r, want, rec, n_rec, faces, L, last_t, last_c, more);
    if (more) cnt.rare(C_OVERFLOW);
    wave_sync();  // the ring may share the staged faces' memory
    int k = 0, steps = 0, head = 0, tail = 0;
    bool fresh = false;  // the entry being walked has no chord of some length yet
    WalkPos w = {};
    w.code = -1;  // no walk in progress
    double tin = 0.0;
    Cutter cut;
    while (true) {
      const bool next = (w.code < 0) & (k < n) & (head == tail) & !cut.cutting();
      if (ballot(next)) steps = 0;
      fresh |= next;
      if (next) {  // the next entry
        start_walk(M, r, L.Cd(k), w, tin, cut.s1);
        cut.start(f, tin, cut.s1);
        ++cnt.entries;
        ++k;
      }
      const WalkRec wr = walk_rec(M, max(w.code, 0));
      const unsigned long long walks = ballot(w.code >= 0), live = walks | ballot(k < n);
      while (true) {  // rounds of one piece per lane
        const unsigned long long act = ballot(cut.cutting()) | ballot(head < tail);
        if (!act || (live && __popcll(act) * 64 < ROUND_LANES * __popcll(act | live) &&
                     !(walks & ballot(tail - head >= CHORDS))))
          break;
        if (!cut.cutting() & (head < tail)) {
          const int slot = (head & (CHORDS - 1)) * WAVE + L.lane;
          cut.to(f, ring.t[slot], ring.s[slot]);
          ++head;
        }
        if (cut.cutting()) {
          float wt, len, s;
          cut.piece(f, wt, len, s);
          sink.piece(wt, len, s);
        }
      }
      if (!live) break;
      const bool alive = w.code >= 0;
      cnt.w_steps += __popcll(walks);
      double tout;
      float sout;
      const bool forward = walk_step(r, w, wr, tin, tout, sout, cnt);
      if (alive) {
        const int slot = (tail & (CHORDS - 1)) * WAVE + L.lane;
        ring.t[slot] = tout;
        ring.s[slot] = sout;
      }
      tail += alive ? 1 : 0;
      cnt.segments += (forward & fresh) ? 1u : 0u;  // a maximal ray interval inside the subdomain
      fresh &= !forward;
      tin = tout;
      if (++steps >= f.max_steps) {  // (every walk has taken at least as many)
        cnt.rare(C_STEPLIMIT, w.code >= 0 ? 1u : 0u);
        w.code = -1;
      }
    }
    if (n > 0) {
      last_t = L.T(n - 1);
      last_c = L.Cd(n - 1);
    }
  }
}

__device__ __forceinline__ unsigned wave_sum(unsigned v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// The wavefront's counts, added to the workgroup's copy of the counters by one instruction (lane c adds counter
// c).  The copies are 128-byte lines of their own and workgroups of one XCD share 8 of them: atomics of all XCDs on
// one line are served one after another, and that bounded the launches with a workgroup per (tile, subdomain)
// pair (stage one, 1024^2, 72 subdomains, m = 4: 2.28 ms with one copy, 1.28 with 64; 512^2, m = 6: 0.69, 0.51).
__device__ __forceinline__ void flush_counts(const LaneCount& c, unsigned long long* ctr) {
  const int lane = threadIdx.x & (WAVE - 1);
  unsigned v = 0u;
  auto put = [&](int which, unsigned sum) { v = lane == which ? sum : v; };
  put(C_PIECES, wave_sum(c.pieces) + c.w_pieces);
  put(C_STEPS, c.w_steps);
  put(C_ENTRIES, wave_sum(c.entries));
  put(C_NONPD, wave_sum(c.nonpd));
  put(C_TABLED, c.w_tabled);
  put(C_TABFB, c.w_fallback);
  put(C_SEGMENTS, wave_sum(c.segments));
  if (v) atomicAdd(ctr + size_t(blockIdx.x % CTR_COPIES) * CTR_STRIDE + lane, (unsigned long long)v);
}

// ------------------------------------------------------------------ stage one

// The moments accumulate in FP64: a ray crosses hundreds of pieces per
// subdomain at the largest workloads, where FP32 sums would drift by ~1e-5 of
// b0; FP64 adds cost the same issue slot as FP32 ones here and need no
// compensation terms.
// A lane's share of the piece store: the chunk it is filling and the pieces
// it kept so far (over all subdomains, in walk order).  Chunks come from a
// block of STORE_BLOCK chunks that the wavefront takes with one atomic; the
// block's state lives in LDS (its lanes diverge, so no register copy of it
// stays current).  One atomic per chunk on a single counter was measured to
// serialise: stage one took 5x as long.
typedef __attribute__((address_space(3))) volatile unsigned long long lds_vu64;
typedef __attribute__((address_space(3))) volatile int lds_vi32;
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long v, int l) {
  const unsigned lo = __builtin_amdgcn_readlane(unsigned(v & 0xffffffffull), l);
  const unsigned hi = __builtin_amdgcn_readlane(unsigned(v >> 32), l);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
struct LaneStore {
  PieceStore ps;
  size_t slot;     // tile * 64 + lane
  unsigned kept;
  float* cur;      // where the next piece goes in the current chunk
  bool keep;
  // LDS: first chunk of the wavefront's block and the chunks of it handed
  // out.  Written by one lane and read by others in later divergent regions,
  // so volatile; LDS-addressed, so a read waits for LDS only (a generic
  // access would also wait for every piece store still in flight).
  lds_vu64* blk_base;
  lds_vi32* blk_used;
  // append one piece; lanes that start a chunk at this point get consecutive
  // chunks of the wavefront's block (and a new block when it runs out)
  __device__ void put(float z, float a, float s, int lane) {
    if (!keep) return;
    if ((kept & (PIECE_CHUNK - 1)) == 0) {
      const unsigned long long need = __ballot(1);
      const int leader = __builtin_ffsll(static_cast<long long>(need)) - 1;
      const int n = __popcll(need);
      const int r = __popcll(need & ((1ull << lane) - 1));
      const unsigned long long base = *blk_base;  // every lane reads the same word
      const int used = *blk_used;
      const int rem = STORE_BLOCK - used;
      unsigned long long fresh = 0;
      if (n > rem) {
        unsigned long long got = 0;
        if (lane == leader) got = atomicAdd(ps.next, (unsigned long long)STORE_BLOCK);
        fresh = readlane_u64(got, leader);
      }
      const unsigned long long id = r < rem ? base + used + r : fresh + (r - rem);
      if (lane == leader) {
        if (n > rem) {
          *blk_base = fresh;
          *blk_used = n - rem;
        } else {
          *blk_used = used + n;
        }
      }
      const unsigned k = kept / PIECE_CHUNK;
      if (id < static_cast<unsigned long long>(ps.n_chunks) && k < unsigned(ps.maxc)) {
        ps.ptab[slot * ps.maxc + k] = int(id);
        cur = ps.pool + size_t(id) * (PIECE_CHUNK * 3);
      } else {
        keep = false;
        atomicAdd(ps.next + 1, 1ull);
        return;
      }
    }
    cur[0] = z;
    cur[1] = a;
    cur[2] = s;
    cur += 3;
    ++kept;
  }
};

// KEEP: stage one also keeps every piece for stage two (the pieces then need
// not be walked again); fixed per launch, so the store costs no registers
// when it is off.
template <int M1, bool KEEP>
struct MomentSink {
  const FrameDev* f;
  const float2* tfa;  // LDS: kappa times the table's alpha column and its differences
  double b[M1];
  unsigned pieces;
  LaneStore st;      // st.keep false: pieces are not kept
  int lane;
  __device__ __forceinline__ void piece(float wt, float len, float s) {
    int i0;
    float fr;
    tf_coord(*f, s, i0, fr);
    const float2 e = tfa[i0];
    const float a = piece_a(*f, fmaf(fr, e.y, e.x), len);
    const double z = piece_z(*f, wt), ad = a;
    b[0] += ad;
    double zj = z;  // Alg. 2: moment j gains absorbance * depth^j
    const double z2 = z * z;
    double zk = z2;
#pragma unroll
    for (int j = 1; j < M1; ++j) {
      b[j] = fma(ad, zj, b[j]);
      const double nx = zj * z2;  // z^(j+2): two chains, odd and even powers
      zj = zk;
      zk = nx;
    }
    if constexpr (KEEP) st.put(float(z), a, s, lane);
    ++pieces;
  }
};

// Waves per SIMD the walk kernels are compiled for (register budget 512 / n).
constexpr int WALK_WAVES = 3;

template <int M1, bool KEEP, bool QUEUE>
__global__ __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(WALK_WAVES, 8))) void k_moments(MeshDev M, FrameDev f,
                                                  const int* __restrict__ offsets, const int* __restrict__ counts,
                                                  const int* __restrict__ records, const float* __restrict__ tf_rgba,
                                                  float* __restrict__ out, double* __restrict__ gacc,
                                                  int* __restrict__ pcount, int* __restrict__ segs, long long bin_cap,
                                                  PieceStore ps, unsigned long long* ctr, int* queue,
                                                  const int* __restrict__ pair_idx, const int* __restrict__ pair_list) {
  extern __shared__ float4 dyn_lds[];
  float2* tfa = reinterpret_cast<float2*>(dyn_lds);  // [n_tf] kappa * alpha and its differences
  __shared__ union {
    FaceL faces[CHUNK];  // while entries are collected: the chord queues are empty then
    ChordRing<CHORDS> ring;
  } sh;
  __shared__ float ent_t[E_MAX * WAVE];
  __shared__ int ent_c[E_MAX * WAVE];
  const int lane = threadIdx.x;
  for (int i = lane; i < f.n_tf; i += WAVE) {
    const float a0 = kappa_alpha(f, tf_rgba[4 * i + 3]), a1 = kappa_alpha(f, tf_rgba[4 * min(i + 1, f.n_tf - 1) + 3]);
    tfa[i] = make_float2(a0, a1 - a0);
  }
  __shared__ unsigned long long blk_base;
  __shared__ int blk_used;
  if (lane == 0) {
    blk_base = 0;
    blk_used = STORE_BLOCK;  // no block yet
  }
  __syncthreads();
  // a pair list (tiles form): this workgroup walks the one (tile, subdomain) pair blockIdx.x names;
  // else every subdomain of its tile
  int k_first = 0, k_end = f.n_slots;
  int tile = QUEUE ? __builtin_amdgcn_readfirstlane(lane == 0 ? queue_take(queue, f.n_tiles) : 0)
                   : xcd_tile(blockIdx.x, gridDim.x);
  if (!QUEUE && pair_list) {
    const int bin = pair_list[blockIdx.x];
    tile = bin / f.n_slots;
    k_first = bin - tile * f.n_slots;
    k_end = k_first + 1;
  }
  for (; tile >= 0;
       tile = QUEUE ? __builtin_amdgcn_readfirstlane(lane == 0 ? queue_take(queue, f.n_tiles) : 0) : -1) {
  const int tx = tile % f.tiles_x, ty = tile / f.tiles_x;
  const int px = (tx << f.tw_log2) + (lane & ((1 << f.tw_log2) - 1)),
            py = ty * (WAVE >> f.tw_log2) + (lane >> f.tw_log2);
  const bool valid = px < f.W && py < f.H;
  const Ray r = pixel_ray(f, valid ? py : 0, valid ? px : 0);
  const size_t HW = size_t(f.W) * f.H, pix = size_t(py) * f.W + px;
  EntryList L{ent_t, ent_c, lane};
  LaneCount cnt = {};
  cnt.ctr = ctr;
  int covering = 0;  // subdomains with at least one piece on this ray
  // the global sum's FP64 partials: in registers at m = 4 (room within the register budget of 3
  // wavefronts per SIMD), else in the per-pixel scratch gacc; the same additions either way
  constexpr bool REG_ACC = M1 <= 5;
  double acc[REG_ACC ? M1 : 1];
  MomentSink<M1, KEEP> sink;  // one sink for all subdomains: its piece store runs across them
  sink.f = &f;
  sink.tfa = tfa;
  sink.st = LaneStore{ps, size_t(tile) * WAVE + lane, 0u, nullptr, ps.pool != nullptr && valid, (lds_vu64*)&blk_base,
                      (lds_vi32*)&blk_used};
  sink.lane = lane;
  for (int k = k_first; k < k_end; ++k) {
    const int bin = tile * f.n_slots + k;
    const int n_rec = counts[bin];
    sink.pieces = 0;
#pragma unroll
    for (int j = 0; j < M1; ++j) sink.b[j] = 0.0;
    if (n_rec > 0 && offsets[bin] + n_rec <= bin_cap) {
      walk_subdomain(M, f, r, valid, records + offsets[bin], n_rec, sh.faces, L, sh.ring, sink, cnt);
    } else if (n_rec > 0) {
      cnt.rare(C_OVERFLOW);  // binned beyond the record capacity (never on an eagerly sized workspace)
    }
    cnt.pieces += sink.pieces;
    if (gacc) {
      // the global sum in slot order, one FP64 partial per pixel: a subdomain without pieces adds an exact
      // zero, so only the others are read and written, and the first one needs no read
      if (valid && sink.pieces > 0) {
        size_t at = pix;
        asm volatile("" : "+v"(at));  // the addresses of the planes are formed here, not kept across the walk
        double* g = gacc + at;
#pragma unroll
        for (int j = 0; j < M1; ++j) {
          const double v = double(float(sink.b[j]));
          if constexpr (REG_ACC)
            acc[j] = covering > 0 ? acc[j] + v : v;
          else
            g[size_t(j) * HW] = covering > 0 ? g[size_t(j) * HW] + v : v;
        }
      }
    } else if (pair_idx) {  // tiles form: only pairs with binned faces, every lane (zeros outside the image)
      if (n_rec > 0) {
        const int p = !QUEUE && pair_list ? int(blockIdx.x) : pair_idx[bin];
        float* o = out + size_t(p) * M1 * WAVE + lane;
#pragma unroll
        for (int j = 0; j < M1; ++j) o[j * WAVE] = float(sink.b[j]);
      }
    } else if (valid) {
      size_t at = pix;
      asm volatile("" : "+v"(at));
      float* o = out + size_t(k) * M1 * HW + at;
#pragma unroll
      for (int j = 0; j < M1; ++j) o[size_t(j) * HW] = float(sink.b[j]);
    }
    covering += sink.pieces > 0 ? 1 : 0;
  }
  if (gacc && valid) {
    size_t at = pix;
    asm volatile("" : "+v"(at));
    float* o = out + at;
#pragma unroll
    for (int j = 0; j < M1; ++j) {
      double t = 0.0;
      if (covering > 0) {
        if constexpr (REG_ACC)
          t = acc[j];
        else
          t = gacc[size_t(j) * HW + at];
      }
      o[size_t(j) * HW] = float(t);
    }
  }
  if (pcount) pcount[size_t(tile) * WAVE + lane] = int(cnt.pieces);
  if (segs && valid) {  // [2][H][W]: segments, covering subdomains
    if (!QUEUE && pair_list) {  // a part of the pixel's, onto zeros
      if (cnt.segments) atomicAdd(segs + pix, int(cnt.segments));
      if (covering) atomicAdd(segs + HW + pix, covering);
    } else {
      segs[pix] = int(cnt.segments);
      segs[HW + pix] = covering;
    }
  }
  flush_counts(cnt, ctr);
  }  // tiles
}

// ------------------------------------------------------------------ stage two, kept pieces
//
// When stage one kept its pieces, stage two evaluates them without a walk:
// one wavefront per tile, a lane per pixel, each lane its pieces in walk order.

__device__ __forceinline__ float4 finalize_px(float4 acc, float b0, int finalize, int renormalize) {
  if (!finalize) return acc;
  if (!renormalize) return acc;
  float A = -expm1f(-b0);
  float sc = acc.w > 1e-30f ? A / acc.w : 0.0f;
  return make_float4(acc.x * sc, acc.y * sc, acc.z * sc, A);
}

// The global moments b_0..b_2N of one pixel (zero for an invalid lane), from
// the FP32 image [2N+1][H][W] or its packed FP16 form [2N+3][H][W] (ln b0 and
// the mean, each as two halves, and the central moments); returns b0 in FP32.
template <int N, class R>
__device__ __forceinline__ float pixel_moments(const void* moments, int f16, bool valid, size_t pix, size_t HW,
                                               R* b) {
  constexpr int M1 = 2 * N + 1;
  float b0f;
  if (f16) {
    const _Float16* hm = static_cast<const _Float16*>(moments);
    const double lb0 = valid ? double(hm[pix]) + double(hm[HW + pix]) : -HUGE_VAL;
    b0f = float(exp(lb0));  // exp(-inf) = 0: background
    double c[M1];
    c[0] = 1.0;
    c[1] = 0.0;
#pragma unroll
    for (int k = 2; k < M1; ++k) c[k] = valid ? double(hm[size_t(k + 2) * HW + pix]) : 0.0;
    const double mu = valid ? double(hm[2 * HW + pix]) + double(hm[3 * HW + pix]) : 0.0;
    b[0] = R(b0f);
#pragma unroll
    for (int j = 1; j < M1; ++j) {  // beta_j = E[z^j] = sum_k C(j, k) mu^(j-k) E[(z - mu)^k]
      double sum = 0.0, binom = 1.0, pw = 1.0;
#pragma unroll
      for (int k = j; k >= 0; --k) {  // term k: C(j, k) c_k mu^(j-k)
        sum += binom * c[k] * pw;
        pw *= mu;
        binom = binom * double(k) / double(j - k + 1);
      }
      b[j] = R(sum * double(b0f));
    }
  } else {
    const float* fm = static_cast<const float*>(moments);
#pragma unroll
    for (int j = 0; j < M1; ++j) b[j] = valid ? R(fm[size_t(j) * HW + pix]) : R(0);
    b0f = valid ? fm[pix] : 0.0f;
  }
  return b0f;
}

// The per-pixel part of Alg. 3, once per pixel instead of once per sample: the bound, its zeros (in LDS, 8
// registers less across the loop over the samples; n >= 3) and an empty continuation.  Returns b0 in FP32.
template <int N, class R, class Z>
__device__ __forceinline__ float pixel_bound(const void* moments, const BoundParams& bp, bool valid, size_t pix,
                                             size_t HW, apcm::Bound<N, R>& bound, const Z& zs,
                                             typename apcm::Bound<N, R>::Cont& cont, LaneCount& cnt) {
  cont.k = -1;
#pragma unroll
  for (int c = 0; c < int(sizeof(cont.v) / sizeof(R)); ++c) cont.v[c] = R(0);
  R b[2 * N + 1], bias[2 * N], zsr[N];
  const float b0f = pixel_moments<N, R>(moments, bp.moments_f16, valid, pix, HW, b);
#pragma unroll
  for (int j = 0; j < 2 * N; ++j) bias[j] = R(bp.bias[j]);
  cnt.nonpd += bound.setup(b, R(bp.alpha), bias, zsr);
  // no zeros found (never expected for a positive definite factor): no shortcut, every sample solves
  if (bound.mode == 2 && !(zsr[0] < zsr[N - 1])) {
    bound.xlo = zsr[0] = -R(HUGE_VAL);
    bound.xhi = zsr[N - 1] = R(HUGE_VAL);
  }
  if constexpr (N >= 3) {
    if (bound.mode != 2) zsr[0] = zsr[N - 1] = __builtin_nan("");  // never continued
#pragma unroll
    for (int i = 0; i < N; ++i) zs[i] = zsr[i];
  }
  return b0f;
}

// Moment bound for every kept piece of a tile and the per-pixel colour sums
// (Alg. 1 second loop, Alg. 3).  A lane takes its pixel's pieces in walk order,
// each with the roots the previous one left (apcm::Bound::frac_continued, n >= 3).
// Bound by FP64 arithmetic at n >= 3, whose few wavefronts re-read their lanes'
// lines from L2; at n = 2 the lanes of all wavefronts hold more lines than L2
// does, so a lane reads four pieces at once (1024^2, m = 4: 2.9 ms one at a
// time, 1.1 now).  The form before took a pixel's pieces 64 at a time, one per
// lane, each from a table of its gaps' roots that the 64 lanes filled with closed
// forms first: a third of the time, and four Newton steps a piece.  Measured,
// 1024^2 on 1.6M tets in 16 subdomains, three views, before and now: m = 8 3.8 to
// 4.1 and 1.9 to 2.3 ms, m = 6 2.7 to 2.9 and 1.7 to 1.9, m = 4 1.16 to 1.27 and
// 1.08 to 1.21.
constexpr int EVAL_WPB = 4;  // wavefronts (tiles) per workgroup: they share the transfer function in LDS

template <int N, class R>
__global__ __launch_bounds__(WAVE * EVAL_WPB) __attribute__((amdgpu_waves_per_eu(N >= 4 ? 3 : 4, 8))) void k_eval(
    FrameDev f, int tile_lo, int tile_hi, PieceStore ps, const int* __restrict__ pcount,
    const float* __restrict__ tf_rgba, const void* __restrict__ moments, BoundParams bp, float* __restrict__ rgba,
    unsigned long long* ctr) {
  extern __shared__ float4 dyn_lds[];
  float4* tf = dyn_lds;  // [n_tf + 1] RGBA
  __shared__ R zs_all[EVAL_WPB][N >= 3 ? N * WAVE : 1];
  for (int i = threadIdx.x; i <= f.n_tf; i += WAVE * EVAL_WPB) {  // (the last entry twice)
    const float* e = tf_rgba + 4 * min(i, f.n_tf - 1);
    tf[i] = make_float4(e[0], e[1], e[2], e[3]);
  }
  __syncthreads();  // the only workgroup barrier
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int tile = tile_lo + xcd_tile(blockIdx.x, gridDim.x, (XCD_RUN + EVAL_WPB - 1) / EVAL_WPB) * EVAL_WPB + wv;
  if (tile >= tile_hi) return;
  const int tx = tile % f.tiles_x, ty = tile / f.tiles_x;
  const int px = (tx << f.tw_log2) + (lane & ((1 << f.tw_log2) - 1)),
            py = ty * (WAVE >> f.tw_log2) + (lane >> f.tw_log2);
  const bool valid = px < f.W && py < f.H;
  const size_t HW = size_t(f.W) * f.H, pix = size_t(py) * f.W + px;
  const size_t slot = size_t(tile) * WAVE + lane;
  // a lane of stage one that could not keep its pieces leaves its chunk table unset: then nothing is read (counted)
  const bool staged = ps.next[1] == 0;
  LaneCount cnt = {};
  cnt.ctr = ctr;
  if (!staged && lane == 0) cnt.rare(C_OVERFLOW);
  apcm::Bound<N, R> bound;
  const apcm::StridedStore<N, R, WAVE> zs{zs_all[wv] + lane};
  typename apcm::Bound<N, R>::Cont cont;
  const float b0f = pixel_bound<N, R>(moments, bp, valid, pix, HW, bound, zs, cont, cnt);
  // (no absorbance on the ray: every piece has a = 0)
  const int np = staged && valid && bound.mode != 0 ? min(pcount[slot], ps.maxc * PIECE_CHUNK) : 0;
  const int* chunks = ps.ptab + slot * size_t(ps.maxc);
  const R eta = R(bp.eta), exponent = bound.b0 * R(-1.4426950408889634074);
  float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
  unsigned solved = 0u, fresh = 0u, closed_used = 0u;
  constexpr int BATCH = N >= 3 ? 1 : 4;  // pieces read at once
  int at = 0;                            // the next batch; read ahead:
  int ahead = np > 0 ? chunks[0] : 0;    // the id of the chunk after the one being read
  const float* chunk = ps.pool;          // the chunk being read
  float next[3 * BATCH] = {};            // z, a, s of each piece
  auto fetch = [&]() {
    if (at >= np) return;
    const int i = at & (PIECE_CHUNK - 1);
    if (i == 0) {
      if (unsigned(ahead) >= unsigned(ps.n_chunks)) {  // cannot happen when every lane kept its pieces; never read
        cnt.rare(C_OVERFLOW);
        ahead = 0;
      }
      chunk = ps.pool + size_t(ahead) * (PIECE_CHUNK * 3);
      ahead = at + PIECE_CHUNK < np ? chunks[at / PIECE_CHUNK + 1] : 0;
    }
#pragma unroll
    for (int k = 0; k < 3 * BATCH; ++k) next[k] = chunk[3 * i + k];  // (a chunk is whole batches)
  };
  static_assert(PIECE_CHUNK % BATCH == 0, "a chunk is whole batches");
  fetch();
  // the colour sums: FP32 over 8 pieces (every lane's at the same time), then FP64
  double sum[4] = {};
  auto flush = [&]() {
    sum[0] += double(a0);
    sum[1] += double(a1);
    sum[2] += double(a2);
    sum[3] += double(a3);
    a0 = a1 = a2 = a3 = 0.0f;
  };
  while (true) {
    R z = R(0);
    float a = 0.0f, fr = 0.0f;
    int i0 = 0;
    auto add = [&](R F, bool now) {  // the piece's colour, weighted
      const float T = fminf(__builtin_amdgcn_exp2f(float(exponent * F)), 1.0f);
      const float w = now ? T * opacity(a) : 0.0f;
      const float4 c0 = tf[i0], c1 = tf[i0 + 1];
      a0 = fmaf(w, fmaf(fr, c1.x - c0.x, c0.x), a0);
      a1 = fmaf(w, fmaf(fr, c1.y - c0.y, c0.y), a1);
      a2 = fmaf(w, fmaf(fr, c1.z - c0.z, c0.z), a2);
      a3 += w;
    };
    bool unsettled = false;
    while (ballot(at < np)) {  // a batch per lane
      if (at < np) {
        float now[3 * BATCH];
#pragma unroll
        for (int k = 0; k < 3 * BATCH; ++k) now[k] = next[k];
        const int left = np - at;
        if ((at & 7) == 0) flush();
        at += BATCH;
        fetch();
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
          if (k > 0 && k >= left) continue;
          z = R(now[3 * k]);
          a = now[3 * k + 1];
          tf_coord(f, now[3 * k + 2], i0, fr);
          R F;
          if constexpr (N >= 3) {
            unsettled = !bound.frac_continued(z, eta, zs, cont, F, solved, fresh);
          } else {
            F = bound.frac_before(z, eta);
          }
          add(F, !unsettled);
        }
      }
      if constexpr (N >= 3) {
        if (ballot(unsettled)) break;
      }
    }
    if constexpr (N >= 3) {
      if (ballot(unsettled)) {  // the closed forms, out of line: not inside the loop
        if (unsettled) {
          add(bound.frac_closed(z, eta, zs, cont), true);
          ++closed_used;
        }
        continue;
      }
    }
    break;
  }
  cnt.w_tabled += wave_sum(solved);
  cnt.w_fallback += wave_sum(closed_used);
  flush();
  if (valid)
    reinterpret_cast<float4*>(rgba)[pix] =
        finalize_px(make_float4(float(sum[0]), float(sum[1]), float(sum[2]), float(sum[3])), b0f, bp.finalize,
                    bp.renormalize);
  flush_counts(cnt, ctr);
}

// ------------------------------------------------------------------ stage two, fused re-walk
//
// The plain form of stage two (Alg. 1 second loop, Section 4.2): every ray is
// walked again exactly like stage one (the same pieces with bit for bit the
// same warped depths and optical depths), and each piece is weighted at once
// by the transmittance the moment bound gives at its depth.  Per pixel nothing
// but (m + 1) moments in and 4 colour sums out, whatever the depth
// complexity; no piece is written to memory.
//
// Each tile is one workgroup of two wavefronts, a walker and an evaluator.
// The walk is bound by its dependent record loads and the evaluation by FP64
// arithmetic, and the evaluation's per-pixel state (inverse Cholesky factor,
// zeros of the degree-n orthonormal polynomial, continuation of the roots) is
// what limits how many wavefronts a SIMD holds.  Split this way neither
// wavefront holds the other's registers, and the evaluator's arithmetic fills
// the issue slots the walker spends waiting on memory.  The chords' ends pass
// through a ring of PQ slots per lane in LDS, and the evaluator cuts them into
// pieces as stage one does (handing over the pieces themselves cost the walker
// a loop over each chord's pieces and the pair 16 bytes a piece).  The two wavefronts meet at phase boundaries
// (workgroup barriers): at each the walker publishes how many chords each lane
// has produced and the evaluator how many it has taken; between two boundaries
// the evaluator takes only chords published at the earlier one and the walker
// writes only ring slots taken before it, so they never touch the same slot.
// Per lane the pieces are evaluated in walk order, each with the roots the
// previous one left (apcm::Bound::frac_continued, n >= 3).  Bound by the
// evaluator's vector instructions: it waits at 5 % of the boundaries' time, the
// walker at 55 %, and two evaluators to a walker were slower (39 ms against 33
// at the largest frame below), as were evaluators and walkers on swapped SIMDs.
// Measured, m = 8: 2560^2 on 12.6M tets 41.8 ms with pieces in the ring, 33.4 now;
// 1024^2 on 1.6M tets in 72 uneven subdomains 5.07, 3.93.
//
// The pair's shape for n = N roots: wavefronts per SIMD the kernel is compiled for (register budget 512 / n),
// slots of the ring (one bit each in half a word) and evaluation rounds (one piece per lane) per phase at most.
// Four wavefronts per SIMD need 128 registers and 20 KB of LDS per workgroup: the bound's state fits for n <= 3
// (but for 3 registers at n = 3 by tiles) with a ring of 8, and a phase there takes about what half the ring holds.  At n = 4 the state does not fit
// (spills in the loop: 83 ms), and a ring of 16 lets the walker run further ahead.  Measured, re-walk ms of the
// 2560^2 frame of a 12.6M-tet mesh at m = 8: 3 wavefronts, ring 16: 33.2 with 12 rounds, 33.4 with 8; ring 8:
// 34.1 with 5; of the 1024^2 frame of a 1.6M-tet mesh at m = 6 and m = 4: 4 wavefronts, ring 8, 5 rounds: 2.56
// and 2.18, 3 wavefronts, ring 16, 8 rounds: 2.84 and 2.59.
template <int N>
struct PairShape {
  static constexpr int WAVES = N >= 4 ? 3 : 4, PQ = N >= 4 ? 16 : 8, ROUNDS = N >= 4 ? 12 : 5;
};

template <int PQ>
struct PairLDS {
  static_assert(PQ <= 16, "one bit per ring slot in tail");
  ChordRing<PQ> ring;
  // the low PQ bits: which slots hold the start of a segment instead of a chord; above them the number of
  // records lane l has produced (mod 2^(32 - PQ)), published at the boundaries of each parity
  unsigned tail[2][WAVE];
  unsigned head[2][WAVE];  // records lane l has taken
  int done[2];             // the walker has no more
};

// The walker's side of the ring.
template <int PQ>
struct Producer {
  PairLDS<PQ>* sh;
  int lane, parity;
  unsigned tail;    // records produced
  unsigned limit;   // slots free up to here (taken count at the last boundary + PQ)
  unsigned starts;  // bit per slot

  __device__ __forceinline__ bool full() const { return tail == limit; }
  __device__ __forceinline__ void put(double t, float s, unsigned start) {
    const unsigned j = tail & (PQ - 1), slot = j * WAVE + lane;
    sh->ring.t[slot] = t;
    sh->ring.s[slot] = s;
    starts = (starts & ~(1u << j)) | (start << j);
    ++tail;
  }
  // phase boundary (the whole walker wavefront): publish, meet the evaluator, learn what it has taken
  __device__ __forceinline__ void boundary(bool finished) {
    sh->tail[parity][lane] = (tail << PQ) | starts;
    if (lane == 0) sh->done[parity] = finished ? 1 : 0;
    __syncthreads();
    limit = sh->head[parity][lane] + PQ;
    parity ^= 1;
  }
};

// All entries of this lane's ray into one subdomain, walked in (depth, code)
// order as in walk_subdomain (same chords, same order).  The wavefront steps
// together; when a lane's ring is full it ends its phase.
template <int PQ>
__device__ void walk_subdomain_paired(const MeshDev& M, const FrameDev& f, const Ray& r, bool valid, const int* rec,
                                      int n_rec, FaceL* faces, EntryList& L, Producer<PQ>& q, LaneCount& cnt) {
  float last_t = -FLT_MAX;
  int last_c = -1;
  bool more = true;
  while (true) {
    const bool want = valid && more;
    if (!__any(want)) break;
    const int n = collect_entries<E_MAX>(M, r, want, rec, n_rec, faces, L, last_t, last_c, more);
    if (more) cnt.rare(C_OVERFLOW);
    int k = 0, steps = 0;
    bool fresh = false;  // the entry being walked has no chord of some length yet
    WalkPos w = {};
    w.code = -1;  // no walk in progress
    double tin = 0.0;
    while (true) {
      const unsigned long long todo = ballot(w.code >= 0) | ballot(k < n);
      if (!todo) break;
      if (todo & ballot(q.full())) {
        q.boundary(false);
        continue;
      }
      const bool next = (w.code < 0) & (k < n);
      if (ballot(next)) steps = 0;
      fresh |= next;
      if (next) {  // the next entry
        float s;
        start_walk(M, r, L.Cd(k), w, tin, s);
        q.put(tin, s, 1);
        ++cnt.entries;
        ++k;
      }
      const WalkRec wr = walk_rec(M, max(w.code, 0));
      const unsigned long long walks = ballot(w.code >= 0);
      while (walks & ballot(q.full())) q.boundary(false);
      const bool alive = w.code >= 0;
      cnt.w_steps += __popcll(walks);
      double tout;
      float sout;
      const bool forward = walk_step(r, w, wr, tin, tout, sout, cnt);
      if (alive) q.put(tout, sout, 0);
      cnt.segments += (forward & fresh) ? 1u : 0u;  // a maximal ray interval inside the subdomain
      fresh &= !forward;
      tin = tout;
      if (++steps >= f.max_steps) {  // (every walk has taken at least as many)
        cnt.rare(C_STEPLIMIT, w.code >= 0 ? 1u : 0u);
        w.code = -1;
      }
    }
    if (n > 0) {
      last_t = L.T(n - 1);
      last_c = L.Cd(n - 1);
    }
  }
}

template <int N, class R, bool QUEUE, bool PAIRS>
__global__ __launch_bounds__(2 * WAVE) __attribute__((amdgpu_waves_per_eu(PairShape<N>::WAVES, 8))) void k_resolve(
    MeshDev M, FrameDev f, const int* __restrict__ offsets, const int* __restrict__ counts, const int* __restrict__ records, long long bin_cap,
    const float* __restrict__ tf_rgba, const void* __restrict__ moments, BoundParams bp, float* __restrict__ rgba,
    unsigned long long* ctr, int* queue, const int* __restrict__ pair_list, float* __restrict__ part) {
  extern __shared__ float4 dyn_lds[];
  float4* tf = dyn_lds;  // [n_tf + 1] RGB and kappa * alpha
  __shared__ FaceL faces[CHUNK];
  __shared__ float ent_t[E_MAX * WAVE];
  __shared__ int ent_c[E_MAX * WAVE];
  constexpr int PQ = PairShape<N>::PQ;
  __shared__ PairLDS<PQ> sh;
  __shared__ R zs_lds[N >= 3 ? N * WAVE : 1];  // per pixel, the zeros of the degree-N orthonormal polynomial
  __shared__ int next_tile;
  for (int i = threadIdx.x; i <= f.n_tf; i += 2 * WAVE) {  // (the last entry twice: the end of an interpolation)
    const float* e = tf_rgba + 4 * min(i, f.n_tf - 1);
    tf[i] = make_float4(e[0], e[1], e[2], kappa_alpha(f, e[3]));
  }
  // PAIRS (a launch over pair_list): this workgroup walks the one (tile, subdomain) pair `pair` and writes
  // its colour sums, unfinalised, to part[pair]; else every subdomain of its tile, into the image
  int pair = 0, k_first = 0, k_end = f.n_slots;
  if constexpr (PAIRS) {
    pair = xcd_tile(blockIdx.x, gridDim.x);
    k_first = pair_list[pair] % f.n_slots;
    k_end = k_first + 1;
  }
  if (threadIdx.x == 0)
    next_tile = QUEUE ? queue_take(queue, f.n_tiles)
                      : PAIRS ? pair_list[pair] / f.n_slots : xcd_tile(blockIdx.x, gridDim.x);
  __syncthreads();
  for (int tile = next_tile; tile >= 0;) {  // the same tiles for both wavefronts of the workgroup
  const bool walker = threadIdx.x < WAVE;
  const int lane = threadIdx.x % WAVE;
  const int tx = tile % f.tiles_x, ty = tile / f.tiles_x;
  const int px = (tx << f.tw_log2) + (lane & ((1 << f.tw_log2) - 1)),
            py = ty * (WAVE >> f.tw_log2) + (lane >> f.tw_log2);
  const bool valid = px < f.W && py < f.H;
  LaneCount cnt = {};
  cnt.ctr = ctr;
  if (walker) {
    const Ray r = pixel_ray(f, valid ? py : 0, valid ? px : 0);
    Producer<PQ> q;
    q.sh = &sh;
    q.lane = lane;
    q.parity = 0;
    q.tail = 0u;
    q.limit = PQ;
    q.starts = 0u;
    EntryList L{ent_t, ent_c, lane};
    for (int k = k_first; k < k_end; ++k) {
      const int bin = tile * f.n_slots + k;
      const int n_rec = counts[bin];
      if (n_rec > 0 && offsets[bin] + n_rec <= bin_cap)
        walk_subdomain_paired(M, f, r, valid, records + offsets[bin], n_rec, faces, L, q, cnt);
      else if (n_rec > 0)
        cnt.rare(C_OVERFLOW);  // binned beyond the record capacity (never on an eagerly sized workspace)
    }
    q.boundary(true);
  } else {
    const size_t HW = size_t(f.W) * f.H, pix = size_t(py) * f.W + px;
    // the bound and the continuation are separate locals (a structure holding a run-time indexed array would live
    // in scratch)
    apcm::Bound<N, R> bound;
    const apcm::StridedStore<N, R, WAVE> zs{zs_lds + lane};
    typename apcm::Bound<N, R>::Cont cont;
    const float b0f = pixel_bound<N, R>(moments, bp, valid, pix, HW, bound, zs, cont, cnt);
    const R eta = R(bp.eta);
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
    unsigned solved = 0u, fresh = 0u;  // samples needing roots; of those, in another gap than the last
    const R exponent = bound.b0 * R(-1.4426950408889634074);
    unsigned head = 0u, ready = 0u, starts = 0u;  // records taken; records to take; which of them are starts
    int parity = 0, n = 0;
    bool fin = false;
    Cutter cut;
    double next_t = 0.0;  // the record at `head`, read ahead (the one before it while none is ready)
    float next_s = 0.0f;
    auto fetch = [&]() {
      const unsigned slot = ((ready > 0u ? head : head - 1u) & (PQ - 1)) * WAVE + lane;
      next_t = sh.ring.t[slot];
      next_s = sh.ring.s[slot];
    };
    // Alg. 1 second loop with Alg. 3's bound, a round of one piece per lane at a time (the next chord where the
    // last is used up), in phases of at most PairShape<N>::ROUNDS.  A lane whose bound did not settle leaves the loop
    // with its piece, and the closed forms, out of line, are called outside it (a call inside would cost the
    // loop half its registers).
    while (true) {
      R z = R(0);
      float a = 0.0f, fr = 0.0f;
      int i0 = 0;
      auto add = [&](R F, bool now) {  // the piece's colour, weighted
        const float T = fminf(__builtin_amdgcn_exp2f(float(exponent * F)), 1.0f);
        const float w = now ? T * opacity(a) : 0.0f;
        asm volatile("" : "+v"(i0));  // the colours are read here, not held in registers across the bound
        const float4 c0 = tf[i0], c1 = tf[i0 + 1];
        a0 = fmaf(w, fmaf(fr, c1.x - c0.x, c0.x), a0);
        a1 = fmaf(w, fmaf(fr, c1.y - c0.y, c0.y), a1);
        a2 = fmaf(w, fmaf(fr, c1.z - c0.z, c0.z), a2);
        a3 += w;
      };
      bool unsettled = false;
      while ((ballot(cut.cutting()) | ballot(ready > 0u)) && (fin || n < PairShape<N>::ROUNDS)) {
        ++n;
        if (!cut.cutting() & (ready > 0u)) {
          if ((starts >> (head & (PQ - 1))) & 1)
            cut.start(f, next_t, next_s);
          else
            cut.to(f, next_t, next_s);
          --ready;
          head += 1u;
        }
        fetch();
        const unsigned long long has = ballot(cut.cutting());
        cnt.w_pieces += __popcll(has);
        if (cut.cutting()) {
          float wt, len, s;
          cut.piece(f, wt, len, s);
          if (bound.mode != 0) {  // (no absorbance on the ray: every piece has a = 0)
            tf_coord(f, s, i0, fr);
            const float ka0 = tf[i0].w, ka1 = tf[i0 + 1].w;
            z = R(piece_z(f, wt));
            R F;
            if constexpr (N >= 3) {
              unsettled = !bound.frac_continued(z, eta, zs, cont, F, solved, fresh);
            } else {
              F = bound.frac_before(z, eta);
            }
            a = piece_a(f, fmaf(fr, ka1 - ka0, ka0), len);  // as stage one
            add(F, !unsettled);
          }
        }
        if constexpr (N >= 3) {
          if (ballot(unsettled)) break;
        }
      }
      if constexpr (N >= 3) {
        if (ballot(unsettled)) {
          if (unsettled) add(bound.frac_closed(z, eta, zs, cont), true);
          continue;
        }
      }
      if (fin) break;
      sh.head[parity][lane] = head;
      __syncthreads();
      starts = sh.tail[parity][lane];
      ready = ((starts >> PQ) - head) & (~0u >> PQ);
      fin = sh.done[parity] != 0;
      parity ^= 1;
      n = 0;
      fetch();
    }
    cnt.w_tabled += wave_sum(solved);
    cnt.w_fallback += wave_sum(fresh);
    if constexpr (PAIRS) {  // [pairs][4][64], every lane
      float* o = part + size_t(pair) * 4 * WAVE + lane;
      o[0] = a0;
      o[WAVE] = a1;
      o[2 * WAVE] = a2;
      o[3 * WAVE] = a3;
    } else if (valid) {
      reinterpret_cast<float4*>(rgba)[pix] =
          finalize_px(make_float4(a0, a1, a2, a3), b0f, bp.finalize, bp.renormalize);
    }
  }
  flush_counts(cnt, ctr);
  if (!QUEUE) break;
  // both wavefronts are done with the tile (and with next_tile): take the next one
  __syncthreads();
  if (threadIdx.x == 0) next_tile = queue_take(queue, f.n_tiles);
  __syncthreads();
  tile = next_tile;
  }  // tiles
}

// Walk records: tet t entered through its face f has 32 bytes at wrec[2 * ((t << 2) | f)] -- vertex f, then for
// the exits at positions 0, 1, 2 (the faces opposite the local vertices f ^ 1, f ^ 3, f ^ 2) the code of the tet
// behind (-1 on the hull or where it belongs to another subdomain), then a word of bits about exit p:
//   2p..2p+1   what to add to the walk's `rot` (mod 3): with k = local index ^ exit face here and there, the next
//              tet numbers the face's vertices by a reflection of {1, 2, 3}; it fixes one k, at position q of the
//              order (1, 3, 2), and rot grows by p - q
//   6+2p..     which vertex of the exit face has the smallest id: 0 vertex f, 1 / 2 the one at position p + 1 / p + 2
//   12+p       whether vertex f has a smaller id than the vertex at position p
// sub_begin [n_sub + 1]: first tet of each subdomain.
__global__ void k_walk_records(const int4* __restrict__ tet, const float4* __restrict__ vert, int64_t n,
                               const int* __restrict__ sub_begin, int n_sub, int4* __restrict__ wrec) {
  const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= 4 * n) return;
  const int t = int(g >> 2), fc = int(g & 3);
  int lo = 0, hi = n_sub;  // the subdomain of t: sub_begin[lo] <= t < sub_begin[lo + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sub_begin[mid] <= t)
      lo = mid;
    else
      hi = mid;
  }
  const int t_lo = sub_begin[lo], t_hi = sub_begin[lo + 1];
  const int4 tv = tet[2 * int64_t(t)], tn = tet[2 * int64_t(t) + 1];
  const int id = sel4(tv, fc);
  unsigned info = 0;
  int out[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const int c = p == 0 ? 1 : (p == 1 ? 3 : 2), c1 = p == 0 ? 3 : (p == 1 ? 2 : 1), c2 = p == 0 ? 2 : (p == 1 ? 1 : 3);
    const int ex = fc ^ c;
    const int i1 = sel4(tv, fc ^ c1), i2 = sel4(tv, fc ^ c2);
    info |= (id < i1 && id < i2 ? 0u : (i1 < i2 ? 1u : 2u)) << (6 + 2 * p);
    info |= (id < sel4(tv, ex) ? 1u : 0u) << (12 + p);
    const int nb = sel4(tn, ex), t2 = nb >> 2;
    out[p] = nb >= 0 && t2 >= t_lo && t2 < t_hi ? nb : -1;
    if (out[p] < 0) continue;
    const int4 w = tet[2 * int64_t(t2)];
    int q = 0;
    for (int k = 1; k < 4; ++k) {
      const int v = sel4(tv, ex ^ k);
      const int l2 = w.x == v ? 0 : (w.y == v ? 1 : (w.z == v ? 2 : 3));
      if ((l2 ^ (nb & 3)) == k) q = k == 1 ? 0 : (k == 3 ? 1 : 2);
    }
    info |= unsigned((p - q + 3) % 3) << (2 * p);
  }
  float4* v = reinterpret_cast<float4*>(wrec + 2 * g);
  *v = vert[id];
  wrec[2 * g + 1] = make_int4(out[0], out[1], out[2], int(info));
}

// ------------------------------------------------------------------ binning

__device__ __forceinline__ void project_px(const FrameDev& f, float4 p, float& col, float& row, bool& ok) {
  const float* Minv = f.minv;
  // solve [dir right down] (l, la, lb)^T = p - eye
  float yx = p.x - f.ex, yy = p.y - f.ey, yz = p.z - f.ez;
  float l = Minv[0] * yx + Minv[1] * yy + Minv[2] * yz;
  float la = Minv[3] * yx + Minv[4] * yy + Minv[5] * yz;
  float lb = Minv[6] * yx + Minv[7] * yy + Minv[8] * yz;
  if (f.proj == 0) {
    col = la - 0.5f;
    row = lb - 0.5f;
    ok = true;
  } else {
    ok = l > 1e-6f;
    float il = 1.0f / l;
    col = la * il + f.half_w - 0.5f;
    row = lb * il + f.half_h - 0.5f;
  }
}

__global__ void k_bin(MeshDev M, FrameDev f, const SlotDev* __restrict__ slots,
                      const int* __restrict__ bface, int* __restrict__ counts, const int* __restrict__ offsets,
                      int* __restrict__ cursors, int* __restrict__ records, int fill, long long rec_cap) {
  const int k = blockIdx.y;
  const SlotDev sl = slots[k];
  const int i = sl.face_begin + blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= sl.face_end) return;
  const int code = bface[i];
  const int t = code >> 2, fc = code & 3;
  const int4 tv = M.tet[2 * t];
  const float4 a = M.vert[sel4(tv, fc ^ 1)];
  const float4 b = M.vert[sel4(tv, fc ^ 2)];
  const float4 c = M.vert[sel4(tv, fc ^ 3)];
  // conservative back-face cull: drop faces every ray crosses outwards
  {
    float ux = b.x - a.x, uy = b.y - a.y, uz = b.z - a.z, vx = c.x - a.x, vy = c.y - a.y, vz = c.z - a.z;
    float nx = uy * vz - uz * vy, ny = uz * vx - ux * vz, nz = ux * vy - uy * vx;
    float nn = sqrtf(nx * nx + ny * ny + nz * nz);
    float gx, gy, gz;
    if (f.proj == 0) {
      gx = f.dx;
      gy = f.dy;
      gz = f.dz;
    } else {
      gx = a.x - f.ex;
      gy = a.y - f.ey;
      gz = a.z - f.ez;
    }
    float gn = sqrtf(gx * gx + gy * gy + gz * gz);
    if (gx * nx + gy * ny + gz * nz > 1e-4f * gn * nn) return;
  }
  float cmin = FLT_MAX, cmax = -FLT_MAX, rmin = FLT_MAX, rmax = -FLT_MAX;
  bool all_ok = true;
  const float4 pts[3] = {a, b, c};
  for (int q = 0; q < 3; ++q) {
    float col, row;
    bool ok;
    project_px(f, pts[q], col, row, ok);
    all_ok = all_ok && ok;
    cmin = fminf(cmin, col);
    cmax = fmaxf(cmax, col);
    rmin = fminf(rmin, row);
    rmax = fmaxf(rmax, row);
  }
  int c0, c1, r0, r1;
  if (!all_ok || !(cmax - cmin < 1e7f) || !(rmax - rmin < 1e7f)) {
    c0 = 0;
    r0 = 0;
    c1 = f.W - 1;
    r1 = f.H - 1;
  } else {
    if (cmax < -2.0f || rmax < -2.0f || cmin > float(f.W) + 1.0f || rmin > float(f.H) + 1.0f) return;
    c0 = max(0, int(floorf(cmin)) - 1);
    r0 = max(0, int(floorf(rmin)) - 1);
    c1 = min(f.W - 1, int(ceilf(cmax)) + 1);
    r1 = min(f.H - 1, int(ceilf(rmax)) + 1);
    if (c0 > c1 || r0 > r1) return;
  }
  const int th = WAVE >> f.tw_log2;
  for (int ty = r0 / th; ty <= r1 / th; ++ty)
    for (int tx = c0 >> f.tw_log2; tx <= (c1 >> f.tw_log2); ++tx) {
      const int bin = (ty * f.tiles_x + tx) * f.n_slots + k;
      if (!fill) {
        atomicAdd(counts + bin, 1);
      } else {
        const unsigned pos = unsigned(offsets[bin] + atomicAdd(cursors + bin, 1));
        if (pos < (unsigned long long)rec_cap) records[pos] = code;  // the walks skip bins beyond the capacity
      }
    }
}

// ------------------------------------------------------------------ sums

__global__ void k_sum_moments(const float* __restrict__ in, int n_slots, const int* __restrict__ order,
                              int64_t elems, float* __restrict__ out) {
  int64_t i = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * 4;
  if (i >= elems) return;
  if (i + 4 <= elems && (elems & 3) == 0) {
    double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    for (int k = 0; k < n_slots; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(in + int64_t(order[k]) * elems + i);
      s0 += v.x;
      s1 += v.y;
      s2 += v.z;
      s3 += v.w;
    }
    *reinterpret_cast<float4*>(out + i) = make_float4(float(s0), float(s1), float(s2), float(s3));
  } else {
    for (int64_t e = i; e < elems && e < i + 4; ++e) {
      double s = 0;
      for (int k = 0; k < n_slots; ++k) s += in[int64_t(order[k]) * elems + e];
      out[e] = float(s);
    }
  }
}

// A bin b = tile * n_slots + slot with binned faces is a pair; pidx[b] numbers them in bin order, and pair_bin
// lists their bins in that order.
__global__ void k_pair_list(const int* __restrict__ counts, int64_t nb, const int* __restrict__ pidx,
                            int* __restrict__ pair_bin, int64_t n_pairs) {
  const int64_t b = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (b < nb && counts[b] > 0 && pidx[b] < n_pairs) pair_bin[pidx[b]] = int(b);
}

// A tile's pairs are contiguous in pair_bin (ascending): the first one with a bin >= first_bin, searched by the
// whole wavefront (64 probes a level: three dependent loads for 200k pairs where a binary search takes 18), and
// how many of them are below first_bin + n_slots.  `first` and `n` are the same in every lane.
__device__ __forceinline__ void tile_pairs(const int* __restrict__ pair_bin, int64_t n_pairs, int64_t first_bin,
                                           int n_slots, int lane, int64_t& first, int64_t& n) {
  int64_t lo = 0, hi = n_pairs;  // every pair before lo is below first_bin, none from hi on
  while (lo < hi) {
    const int64_t step = (hi - lo + WAVE - 1) / WAVE, at = lo + lane * step;
    const int c = __popcll(ballot(at < hi && pair_bin[at] < first_bin));  // probes 0 .. c-1 are below
    hi = c < WAVE ? min(hi, lo + c * step) : hi;
    lo = c > 0 ? lo + (c - 1) * step + 1 : hi;
  }
  first = lo;
  n = 0;
  for (int got = WAVE; got == WAVE; n += got) {
    const int64_t at = first + n + lane;
    got = __popcll(ballot(at < n_pairs && pair_bin[at] < first_bin + n_slots));
  }
}

constexpr int SUM_WPB = 4;  // wavefronts (tiles) per workgroup of the two sums below

// Global moments from the tiles form: pixel (tile t, lane l) adds, for the pairs of tile t in slot order
// (ascending subdomain ids), tile p's value at lane l in FP64 -- the additions of k_sum_moments without the
// pairs' zeros (adding an exact 0 changes nothing), so the result is bitwise the dense form's.  A wavefront
// per tile: the search is shared, the reads are whole 256-byte rows, and the sums stay in registers (M1 is
// fixed).  Bound by the latency of its few dependent loads.  Measured, 256^2 / 1024^2 frames of 72 subdomains,
// a thread per pixel with a binary search each and the sums in scratch memory: 86 / 74 us; now 11 / 28 us.
template <int M1>
__global__ __launch_bounds__(WAVE * SUM_WPB) void k_sum_tiles(const float* __restrict__ tiles,
                                                              const int* __restrict__ pair_bin, int64_t n_pairs,
                                                              int n_slots, int W, int H, int tw_log2, int tiles_x,
                                                              int64_t n_tiles, float* __restrict__ out) {
  const int64_t tile = flat_block() * SUM_WPB + __builtin_amdgcn_readfirstlane(int(threadIdx.x / WAVE));
  if (tile >= n_tiles) return;
  const int lane = threadIdx.x % WAVE;
  int64_t first, n;
  tile_pairs(pair_bin, n_pairs, tile * n_slots, n_slots, lane, first, n);
  double acc[M1];
#pragma unroll
  for (int j = 0; j < M1; ++j) acc[j] = 0.0;
  const float* t = tiles + first * (M1 * WAVE) + lane;
#pragma unroll 2
  for (int64_t p = 0; p < n; ++p, t += M1 * WAVE) {
#pragma unroll
    for (int j = 0; j < M1; ++j) acc[j] += double(t[j * WAVE]);
  }
  const int x = int(tile % tiles_x) * (1 << tw_log2) + (lane & ((1 << tw_log2) - 1));
  const int64_t y = tile / tiles_x * (WAVE >> tw_log2) + (lane >> tw_log2);
  if (x >= W || y >= H) return;
  float* o = out + y * W + x;
#pragma unroll
  for (int j = 0; j < M1; ++j) o[int64_t(j) * W * H] = float(acc[j]);
}

// FP16 moment image, planes [m+3][pixels]: ln b0 (-inf on background) and the mean depth mu = beta_1, each as
// two FP16 halves (hi, and the rest lo); the central moments E[(z - mu)^k] (mu = hi + lo), k = 2..m.  Central
// moments keep the spread of a concentrated depth distribution at FP16's relative precision, which raw moments
// (all near mu^j) lose; the split ln b0 keeps the opacity 1 - exp(-b0) near FP32 precision.
__global__ void k_pack_f16(const float* __restrict__ in, int m1, int64_t pixels, _Float16* __restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= pixels) return;
  const float b0 = in[i];
  const bool bg = !(b0 > 0.0f);
  const double lb0 = bg ? 0.0 : log(double(b0));
  const _Float16 lhi = _Float16(lb0);
  out[i] = bg ? _Float16(-HUGE_VALF) : lhi;
  out[pixels + i] = bg ? _Float16(0.0f) : _Float16(lb0 - double(lhi));
  const double inv = bg ? 0.0 : 1.0 / double(b0);
  double beta[9];
  beta[0] = 1.0;
  for (int j = 1; j < m1; ++j) beta[j] = double(in[int64_t(j) * pixels + i]) * inv;
  const _Float16 hi = _Float16(beta[1]);
  const _Float16 lo = _Float16(beta[1] - double(hi));
  const double mu = double(hi) + double(lo);
  out[2 * pixels + i] = bg ? _Float16(0.0f) : hi;
  out[3 * pixels + i] = bg ? _Float16(0.0f) : lo;
  for (int k = 2; k < m1; ++k) {
    // E[(z - mu)^k] = sum_i C(k, i) (-mu)^(k-i) beta_i, Horner in (-mu) with running binomials
    double c = 0.0, binom = 1.0, pw = 1.0;
    for (int t = k; t >= 0; --t) {  // term t: C(k, t) beta_t (-mu)^(k-t)
      c += binom * beta[t] * pw;
      pw *= -mu;
      binom = binom * double(t) / double(k - t + 1);
    }
    out[int64_t(k + 2) * pixels + i] = bg ? _Float16(0.0f) : _Float16(c);
  }
}

// Stage two by pairs: pixel (tile t, lane l) adds the colour sums of tile t's pairs at lane l in slot order
// (ascending subdomain ids) in FP64, then finalises with its b0 (FP32 moment image plane 0) -- the
// per-subdomain partial images' canonical sum, taken over the pairs only (a subdomain without a pair on
// the tile has no piece there).  A wavefront per tile, as k_sum_tiles.
__global__ __launch_bounds__(WAVE * SUM_WPB) void k_sum_color_tiles(const float* __restrict__ part,
                                                                    const int* __restrict__ pair_bin,
                                                                    int64_t n_pairs, int n_slots, int W, int H,
                                                                    int tw_log2, int tiles_x, int64_t n_tiles,
                                                                    const float* __restrict__ b0, BoundParams bp,
                                                                    float4* __restrict__ out) {
  const int64_t tile = flat_block() * SUM_WPB + __builtin_amdgcn_readfirstlane(int(threadIdx.x / WAVE));
  if (tile >= n_tiles) return;
  const int lane = threadIdx.x % WAVE;
  int64_t first, n;
  tile_pairs(pair_bin, n_pairs, tile * n_slots, n_slots, lane, first, n);
  double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
  const float* t = part + first * (4 * WAVE) + lane;
#pragma unroll 2
  for (int64_t p = 0; p < n; ++p, t += 4 * WAVE) {
    s0 += t[0];
    s1 += t[WAVE];
    s2 += t[2 * WAVE];
    s3 += t[3 * WAVE];
  }
  const int x = int(tile % tiles_x) * (1 << tw_log2) + (lane & ((1 << tw_log2) - 1));
  const int64_t y = tile / tiles_x * (WAVE >> tw_log2) + (lane >> tw_log2);
  if (x >= W || y >= H) return;
  const int64_t i = y * W + x;
  out[i] = finalize_px(make_float4(float(s0), float(s1), float(s2), float(s3)), b0[i], bp.finalize, bp.renormalize);
}

__global__ void k_sum_images(const float4* __restrict__ in, int n_slots, const int* __restrict__ order,
                             int64_t pixels, const float* __restrict__ b0, BoundParams bp,
                             float4* __restrict__ out) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= pixels) return;
  double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
  for (int k = 0; k < n_slots; ++k) {
    const float4 v = in[int64_t(order[k]) * pixels + i];
    s0 += v.x;
    s1 += v.y;
    s2 += v.z;
    s3 += v.w;
  }
  out[i] = finalize_px(make_float4(float(s0), float(s1), float(s2), float(s3)), b0[i], 1, bp.renormalize);
}

// ------------------------------------------------------------------ scan / fill

constexpr int SCAN_THREADS = 256, SCAN_ITEMS = 8, SCAN_TILE = SCAN_THREADS * SCAN_ITEMS, SCAN_DIRECT = 8192;

// The bins' scan: where each bin's records start (the exclusive sums of the counts) and the numbers of the bins
// that have any (the pairs), with the fill pass's cursors cleared on the way.  Two launches: the sums of each
// SCAN_TILE bins, then every workgroup adds up the sums before its own (a few thousand words from L2 at the
// largest frames) and scans its bins.  A scan of the counts, one of the pair flags, the clearing and the copies
// of their last elements to the host took 9 launches and 4 copies; a small frame's time is its launches (binning
// of a 128^2 frame of 4 subdomains 75 -> 32 us, of a 256^2 frame of 72 by pairs, its pairs' scan included, 220 ->
// 102 us).
// sums[w]: records of workgroup w's bins << 12 | its pairs (at most SCAN_TILE).
__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ __forceinline__ void load_bins(const int* __restrict__ counts, int64_t at, int64_t nb, int v[SCAN_ITEMS]) {
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) v[k] = at + k < nb ? counts[at + k] : 0;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_bin_sums(const int* __restrict__ counts, int64_t nb,
                                                           unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long part[SCAN_THREADS / WAVE];
  int v[SCAN_ITEMS];
  load_bins(counts, int64_t(blockIdx.x) * SCAN_TILE + threadIdx.x * SCAN_ITEMS, nb, v);
  unsigned long long t = 0;
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) t += (static_cast<unsigned long long>(v[k]) << 12) + (v[k] > 0 ? 1 : 0);
  t = wave_sum64(t);
  if (threadIdx.x % WAVE == 0) part[threadIdx.x / WAVE] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < SCAN_THREADS / WAVE; ++w) t += part[w];
    sums[blockIdx.x] = t;
  }
}

// supers[i]: records of the workgroups from i * SCAN_TILE on << 24 | their pairs (at most SCAN_TILE^2)
__global__ __launch_bounds__(SCAN_THREADS) void k_bin_supers(const unsigned long long* __restrict__ sums, int64_t n,
                                                             unsigned long long* __restrict__ supers) {
  __shared__ unsigned long long part[SCAN_THREADS / WAVE];
  unsigned long long t = 0;
  for (int k = threadIdx.x; k < SCAN_TILE; k += SCAN_THREADS) {
    const int64_t at = int64_t(blockIdx.x) * SCAN_TILE + k;
    const unsigned long long v = at < n ? sums[at] : 0;
    t += ((v >> 12) << 24) + (v & 0xfffu);
  }
  t = wave_sum64(t);
  if (threadIdx.x % WAVE == 0) part[threadIdx.x / WAVE] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < SCAN_THREADS / WAVE; ++w) t += part[w];
    supers[blockIdx.x] = t;
  }
}

// supers, offsets and cursors, pidx, totals (records, pairs): each may be null
__global__ __launch_bounds__(SCAN_THREADS) void k_bin_scan(const int* __restrict__ counts, int64_t nb,
                                                           const unsigned long long* __restrict__ sums,
                                                           const unsigned long long* __restrict__ supers,
                                                           int* __restrict__ offsets, int* __restrict__ cursors,
                                                           int* __restrict__ pidx,
                                                           unsigned long long* __restrict__ totals) {
  constexpr int WAVES = SCAN_THREADS / WAVE;
  __shared__ unsigned long long prec[WAVES], ppair[WAVES], part[WAVES];
  const int lane = threadIdx.x % WAVE, wv = threadIdx.x / WAVE;
  const int64_t at = int64_t(blockIdx.x) * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  int v[SCAN_ITEMS];
  load_bins(counts, at, nb, v);
  unsigned long long rec = 0, pairs = 0;  // before this workgroup's bins
  const unsigned whole = supers ? blockIdx.x / SCAN_TILE : 0u;
  for (unsigned w = threadIdx.x; w < whole; w += SCAN_THREADS) {
    rec += supers[w] >> 24;
    pairs += supers[w] & 0xffffffu;
  }
  for (unsigned w = whole * SCAN_TILE + threadIdx.x; w < blockIdx.x; w += SCAN_THREADS) {
    rec += sums[w] >> 12;
    pairs += sums[w] & 0xfffu;
  }
  rec = wave_sum64(rec);
  pairs = wave_sum64(pairs);
  unsigned long long mine = 0;
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) mine += (static_cast<unsigned long long>(v[k]) << 12) + (v[k] > 0 ? 1 : 0);
  unsigned long long run = mine;  // inclusive over the wavefront's lanes
  for (int o = 1; o < WAVE; o <<= 1) {
    const unsigned long long up = __shfl_up(run, o, WAVE);
    run += lane >= o ? up : 0;
  }
  if (lane == WAVE - 1) part[wv] = run;
  if (lane == 0) {
    prec[wv] = rec;
    ppair[wv] = pairs;
  }
  __syncthreads();
  rec = pairs = 0;
  for (int w = 0; w < WAVES; ++w) {
    rec += prec[w];
    pairs += ppair[w];
    run += w < wv ? part[w] : 0;
  }
  run -= mine;
  rec += run >> 12;
  pairs += run & 0xfffu;
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    if (at + k < nb) {
      if (offsets) {
        offsets[at + k] = int(rec);
        cursors[at + k] = 0;
      }
      if (pidx) pidx[at + k] = int(pairs);
    }
    rec += unsigned(v[k]);
    pairs += v[k] > 0 ? 1 : 0;
  }
  if (totals && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_THREADS - 1) {
    totals[0] = rec;
    totals[1] = pairs;
  }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_local(const int* __restrict__ in, int* __restrict__ out,
                                                             int64_t n, int* __restrict__ sums) {
  __shared__ int part[SCAN_THREADS];
  const int64_t base = int64_t(blockIdx.x) * SCAN_TILE + int64_t(threadIdx.x) * SCAN_ITEMS;
  int v[SCAN_ITEMS];
  int tot = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    v[k] = base + k < n ? in[base + k] : 0;
    tot += v[k];
  }
  part[threadIdx.x] = tot;
  __syncthreads();
  for (int o = 1; o < SCAN_THREADS; o <<= 1) {  // Hillis-Steele inclusive scan
    int add = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
    __syncthreads();
    part[threadIdx.x] += add;
    __syncthreads();
  }
  int run = part[threadIdx.x] - tot;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == SCAN_THREADS - 1) sums[blockIdx.x] = part[threadIdx.x];
}

__global__ void k_scan_add(int* __restrict__ out, int64_t n, const int* __restrict__ sums) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] += sums[i / SCAN_TILE];
}

__global__ void k_fill(int* p, int v, int64_t n) {
  const int64_t i = flat_block() * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Per-subdomain images [n_slots][m1][H][W] that pairs write: zeros at the pixels of the tiles without a pair (the
// pairs write the others), a thread per pixel of a slot.  Bound by its writes.
constexpr int CLEAR_THREADS = 256;
__global__ __launch_bounds__(CLEAR_THREADS) void k_clear_unpaired(const int* __restrict__ counts, int n_slots, int m1,
                                                                  int W, int64_t HW, int tw_log2, int tiles_x,
                                                                  int64_t chunks, float* __restrict__ out) {
  const int64_t b = flat_block(), slot = b / chunks;
  if (slot >= n_slots) return;
  const int64_t pix = (b - slot * chunks) * CLEAR_THREADS + threadIdx.x;
  if (pix >= HW) return;
  const unsigned y = unsigned(pix) / unsigned(W), x = unsigned(pix) - y * unsigned(W);  // (HW <= 2^30)
  const int64_t tile = int64_t(y >> (6 - tw_log2)) * tiles_x + (x >> tw_log2);
  if (counts[tile * n_slots + slot] > 0) return;
  float* o = out + slot * m1 * HW + pix;
  for (int j = 0; j < m1; ++j, o += HW) *o = 0.0f;
}

// ------------------------------------------------------------------ mesh residency

__global__ void k_inc_count(const int4* __restrict__ tv, int64_t n_tets, int* __restrict__ counts) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_tets) return;
  const int4 v = tv[t];
  atomicAdd(counts + v.x, 1);
  atomicAdd(counts + v.y, 1);
  atomicAdd(counts + v.z, 1);
  atomicAdd(counts + v.w, 1);
}

__global__ void k_inc_fill(const int4* __restrict__ tv, int64_t n_tets, const int* __restrict__ offsets,
                           int* __restrict__ cursors, int* __restrict__ inc) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_tets) return;
  const int4 v = tv[t];
  inc[offsets[v.x] + atomicAdd(cursors + v.x, 1)] = int(t);
  inc[offsets[v.y] + atomicAdd(cursors + v.y, 1)] = int(t);
  inc[offsets[v.z] + atomicAdd(cursors + v.z, 1)] = int(t);
  inc[offsets[v.w] + atomicAdd(cursors + v.w, 1)] = int(t);
}

// neighbour of every (tet, face): the other tet holding the face's 3 vertices
__global__ void k_adjacency(const int4* __restrict__ tv, int64_t n_tets, const int* __restrict__ offsets,
                            const int* __restrict__ inc, int* __restrict__ nbr, int* __restrict__ err) {
  const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= 4 * n_tets) return;
  const int t = int(g >> 2), fc = int(g & 3);
  const int4 v = tv[t];
  int f3[3], q = 0;
  for (int k = 0; k < 4; ++k)
    if (k != fc) f3[q++] = sel4(v, k);
  int a = min(f3[0], min(f3[1], f3[2]));
  int found = -1, n_found = 0;
  for (int p = offsets[a]; p < offsets[a + 1]; ++p) {
    const int t2 = inc[p];
    if (t2 == t) continue;
    const int4 w = tv[t2];
    int hit = 0, miss = -1;
    for (int k = 0; k < 4; ++k) {
      const int x = sel4(w, k);
      if (x == f3[0] || x == f3[1] || x == f3[2])
        ++hit;
      else
        miss = k;
    }
    if (hit == 3) {
      found = (t2 << 2) | miss;
      ++n_found;
    }
  }
  if (n_found > 1) atomicOr(err, 1);
  nbr[g] = n_found == 1 ? found : -1;
}

inline unsigned grid1(int64_t n, int b) { return unsigned((n + b - 1) / b); }
// At least n blocks of up to 1024 threads (flat_block; the last ones may have nothing to do) as rows, since a launch
// takes fewer than 2^32 threads in each dimension.
inline dim3 wide_grid(int64_t n) {
  const int64_t x = n < (1 << 20) ? n : (1 << 20);
  return dim3(unsigned(x), unsigned((n + x - 1) / x));
}

}  // namespace

// ------------------------------------------------------------------ launchers

hipError_t launch_bin_count(const MeshDev& m, const FrameDev& f, const SlotDev* slots, int max_faces,
                            const int* bface, int* counts, hipStream_t s) {
  if (max_faces <= 0 || f.n_slots <= 0) return hipSuccess;
  dim3 grid(grid1(max_faces, 256), f.n_slots);
  hipLaunchKernelGGL(k_bin, grid, dim3(256), 0, s, m, f, slots, bface, counts, (const int*)nullptr, (int*)nullptr,
                     (int*)nullptr, 0, 0ll);
  return hipGetLastError();
}

hipError_t launch_bin_fill(const MeshDev& m, const FrameDev& f, const SlotDev* slots, int max_faces,
                           const int* bface, const int* offsets, int* cursors, int* records, long long rec_cap,
                           hipStream_t s) {
  if (max_faces <= 0 || f.n_slots <= 0) return hipSuccess;
  dim3 grid(grid1(max_faces, 256), f.n_slots);
  hipLaunchKernelGGL(k_bin, grid, dim3(256), 0, s, m, f, slots, bface, (int*)nullptr, offsets, cursors, records,
                     1, rec_cap);
  return hipGetLastError();
}

// Workgroups of `kernel` the device holds at once (the grid of a persistent launch), at least one.
template <class K>
static int resident_blocks(K kernel, int block, size_t lds) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, lds) != hipSuccess)
    return 1;
  return cus * per_cu > 0 ? cus * per_cu : 1;
}

// the 8 per-XCD tile counters of a persistent launch start at zero (a fill kernel, not a memset: the
// launch may be captured in a graph)
static hipError_t reset_queue(int* queue, hipStream_t s) {
  hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, s, queue, 0, int64_t(QUEUE_INTS));
  return hipGetLastError();
}

hipError_t launch_moments(int mm, const MeshDev& m, const FrameDev& f, const int* offsets,
                          const int* counts, const int* records, long long bin_cap, const float* tf_rgba, float* out,
                          double* gacc, int* pcount, int* segs, const PieceStore& store,
                          unsigned long long* counters, int* queue, const int* pair_idx, const int* pair_list,
                          int64_t n_pairs, hipStream_t s) {
  const size_t lds = size_t(f.n_tf) * sizeof(float2);
  const dim3 block(WAVE);
  if (pair_list) {
    queue = nullptr;  // a workgroup per pair
    if (n_pairs <= 0) return hipSuccess;
  }
  const dim3 grid(pair_list ? unsigned(n_pairs) : unsigned(f.n_tiles));
  if (queue) {
    const hipError_t e = reset_queue(queue, s);
    if (e != hipSuccess) return e;
  }
#define APC_LAUNCH_MOMENTS_K(M1, KP)                                                                    \
  do {                                                                                                  \
    if (queue)                                                                                          \
      hipLaunchKernelGGL((k_moments<M1, KP, true>), dim3(resident_blocks(k_moments<M1, KP, true>, WAVE, lds)), \
                         block, lds, s, m, f, offsets, counts, records, tf_rgba, out, gacc, pcount, \
                         segs, bin_cap, store, counters, queue, pair_idx, nullptr);                     \
    else                                                                                                \
      hipLaunchKernelGGL((k_moments<M1, KP, false>), grid, block, lds, s, m, f, offsets, counts,   \
                         records, tf_rgba, out, gacc, pcount, segs, bin_cap, store, counters, queue, pair_idx, \
                         pair_list);                                                                    \
  } while (0)
#define APC_LAUNCH_MOMENTS(M1)                                                                          \
  do {                                                                                                  \
    if (store.pool)                                                                                     \
      APC_LAUNCH_MOMENTS_K(M1, true);                                                                   \
    else                                                                                                \
      APC_LAUNCH_MOMENTS_K(M1, false);                                                                  \
  } while (0)
  if (mm == 4)
    APC_LAUNCH_MOMENTS(5);
  else if (mm == 6)
    APC_LAUNCH_MOMENTS(7);
  else
    APC_LAUNCH_MOMENTS(9);
#undef APC_LAUNCH_MOMENTS
#undef APC_LAUNCH_MOMENTS_K
  return hipGetLastError();
}

hipError_t launch_eval(int mm, const FrameDev& f, int tile_lo, int tile_hi, const PieceStore& store,
                       const int* pcount, const float* tf_rgba, const void* moments, const BoundParams& bp,
                       float* rgba, unsigned long long* counters, hipStream_t s) {
  if (tile_hi <= tile_lo) return hipSuccess;
  const size_t lds = size_t(f.n_tf + 1) * sizeof(float4);
  const dim3 grid((tile_hi - tile_lo + EVAL_WPB - 1) / EVAL_WPB), block(WAVE * EVAL_WPB);
  if (mm == 4)
    hipLaunchKernelGGL((k_eval<2, float>), grid, block, lds, s, f, tile_lo, tile_hi, store, pcount, tf_rgba, moments,
                       bp, rgba, counters);
  else if (mm == 6)
    hipLaunchKernelGGL((k_eval<3, double>), grid, block, lds, s, f, tile_lo, tile_hi, store, pcount, tf_rgba,
                       moments, bp, rgba, counters);
  else
    hipLaunchKernelGGL((k_eval<4, double>), grid, block, lds, s, f, tile_lo, tile_hi, store, pcount, tf_rgba,
                       moments, bp, rgba, counters);
  return hipGetLastError();
}

hipError_t launch_resolve(int mm, const MeshDev& m, const FrameDev& f, const int* offsets,
                          const int* counts, const int* records, long long bin_cap, const float* tf_rgba,
                          const void* moments, const BoundParams& bp, float* rgba, unsigned long long* counters,
                          int* queue, const int* pair_list, float* part, int64_t n_pairs, hipStream_t s) {
  const size_t lds = size_t(f.n_tf + 1) * sizeof(float4);
  const dim3 block(2 * WAVE);  // a tile (or a pair) per workgroup at a time: its walker and its evaluator
  if (pair_list) {
    queue = nullptr;
    if (n_pairs <= 0) return hipSuccess;
  }
  const dim3 grid(pair_list ? unsigned(n_pairs) : unsigned(f.n_tiles));
  if (queue) {
    const hipError_t e = reset_queue(queue, s);
    if (e != hipSuccess) return e;
  }
#define APC_LAUNCH_RESOLVE(N, R)                                                                               \
  do {                                                                                                         \
    if (pair_list)                                                                                             \
      hipLaunchKernelGGL((k_resolve<N, R, false, true>), grid, block, lds, s, m, f, offsets, counts,   \
                         records, bin_cap, tf_rgba, moments, bp, rgba, counters, nullptr, pair_list, part);   \
    else if (queue)                                                                                            \
      hipLaunchKernelGGL((k_resolve<N, R, true, false>),                                                      \
                         dim3(resident_blocks(k_resolve<N, R, true, false>, 2 * WAVE, lds)), block, lds, s, m, \
                         f, offsets, counts, records, bin_cap, tf_rgba, moments, bp, rgba, counters,    \
                         queue, nullptr, nullptr);                                                             \
    else                                                                                                       \
      hipLaunchKernelGGL((k_resolve<N, R, false, false>), grid, block, lds, s, m, f, offsets, counts,  \
                         records, bin_cap, tf_rgba, moments, bp, rgba, counters, nullptr, nullptr, nullptr);  \
  } while (0)
  if (mm == 4)
    APC_LAUNCH_RESOLVE(2, float);
  else if (mm == 6)
    APC_LAUNCH_RESOLVE(3, double);
  else
    APC_LAUNCH_RESOLVE(4, double);
#undef APC_LAUNCH_RESOLVE
  return hipGetLastError();
}

hipError_t launch_pack_f16(const float* in, int m1, int64_t pixels, void* out_f16, hipStream_t s) {
  if (pixels <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_f16, dim3(grid1(pixels, 256)), dim3(256), 0, s, in, m1, pixels,
                     static_cast<_Float16*>(out_f16));
  return hipGetLastError();
}

hipError_t launch_walk_records(const int4* tet, const float4* vert, int64_t n_tets, const int* sub_begin, int n_sub,
                               int4* wrec, hipStream_t s) {
  if (n_tets <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_walk_records, dim3(grid1(4 * n_tets, 256)), dim3(256), 0, s, tet, vert, n_tets, sub_begin,
                     n_sub, wrec);
  return hipGetLastError();
}

hipError_t launch_sum_moments(const float* in, int n_slots, const int* order, int64_t elems, float* out,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_sum_moments, dim3(grid1((elems + 3) / 4, 256)), dim3(256), 0, s, in, n_slots, order, elems,
                     out);
  return hipGetLastError();
}

hipError_t launch_bin_scan(const int* counts, int64_t nb, int* offsets, int* cursors, int* pidx, int* tmp,
                           unsigned long long* totals, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(tmp);
  const dim3 grid(grid1(nb, SCAN_TILE)), block(SCAN_THREADS);
  hipLaunchKernelGGL(k_bin_sums, grid, block, 0, s, counts, nb, sums);
  unsigned long long* supers = nullptr;
  if (grid.x > SCAN_DIRECT) {
    supers = sums + grid.x;
    hipLaunchKernelGGL(k_bin_supers, dim3(grid1(grid.x, SCAN_TILE)), block, 0, s, sums, int64_t(grid.x), supers);
  }
  hipLaunchKernelGGL(k_bin_scan, grid, block, 0, s, counts, nb, sums, supers, offsets, cursors, pidx, totals);
  return hipGetLastError();
}

hipError_t launch_pair_list(const int* counts, int64_t nb, const int* pidx, int* pair_bin, int64_t n_pairs,
                            hipStream_t s) {
  if (nb <= 0 || n_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_list, dim3(grid1(nb, 256)), dim3(256), 0, s, counts, nb, pidx, pair_bin, n_pairs);
  return hipGetLastError();
}

hipError_t launch_sum_tiles(const float* tiles, const int* pair_bin, int64_t n_pairs, int n_slots, int m1, int W,
                            int H, int tw_log2, float* out, hipStream_t s) {
  const int tw = 1 << tw_log2, th = WAVE >> tw_log2;
  const int tiles_x = int((int64_t(W) + tw - 1) / tw);
  const int64_t n_tiles = (int64_t(H) + th - 1) / th * tiles_x;
  if (n_tiles <= 0) return hipSuccess;
  const dim3 grid = wide_grid((n_tiles + SUM_WPB - 1) / SUM_WPB), block(WAVE * SUM_WPB);
  if (m1 == 5)
    hipLaunchKernelGGL((k_sum_tiles<5>), grid, block, 0, s, tiles, pair_bin, n_pairs, n_slots, W, H, tw_log2, tiles_x,
                       n_tiles, out);
  else if (m1 == 7)
    hipLaunchKernelGGL((k_sum_tiles<7>), grid, block, 0, s, tiles, pair_bin, n_pairs, n_slots, W, H, tw_log2, tiles_x,
                       n_tiles, out);
  else
    hipLaunchKernelGGL((k_sum_tiles<9>), grid, block, 0, s, tiles, pair_bin, n_pairs, n_slots, W, H, tw_log2, tiles_x,
                       n_tiles, out);
  return hipGetLastError();
}

hipError_t launch_sum_color_tiles(const float* part, const int* pair_bin, int64_t n_pairs, int n_slots, int W, int H,
                                 int tw_log2, const float* b0, const BoundParams& bp, float* out, hipStream_t s) {
  const int tw = 1 << tw_log2, th = WAVE >> tw_log2;
  const int tiles_x = int((int64_t(W) + tw - 1) / tw);
  const int64_t n_tiles = (int64_t(H) + th - 1) / th * tiles_x;
  if (n_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sum_color_tiles, wide_grid((n_tiles + SUM_WPB - 1) / SUM_WPB), dim3(WAVE * SUM_WPB), 0, s,
                     part, pair_bin, n_pairs, n_slots, W, H, tw_log2, tiles_x, n_tiles, b0, bp,
                     reinterpret_cast<float4*>(out));
  return hipGetLastError();
}

hipError_t launch_sum_images(const float* in, int n_slots, const int* order, int64_t pixels, const float* b0,
                             const BoundParams& bp, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_images, dim3(grid1(pixels, 256)), dim3(256), 0, s, reinterpret_cast<const float4*>(in),
                     n_slots, order, pixels, b0, bp, reinterpret_cast<float4*>(out));
  return hipGetLastError();
}

int64_t scan_tmp_elems(int64_t n) {
  int64_t total = 0;
  while (n > 1) {
    n = (n + SCAN_TILE - 1) / SCAN_TILE;
    total += 2 * n + 1;
  }
  return total < 1 ? 2 : total + 1;
}

hipError_t launch_exclusive_scan(const int* in, int* out, int64_t n, int* tmp, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
  int* sums = tmp;
  int* sums_scan = tmp + nb;
  hipLaunchKernelGGL(k_scan_local, dim3(unsigned(nb)), dim3(SCAN_THREADS), 0, s, in, out, n, sums);
  if (nb > 1) {
    hipError_t e = launch_exclusive_scan(sums, sums_scan, nb, tmp + 2 * nb + 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3(grid1(n, 256)), dim3(256), 0, s, out, n, (const int*)sums_scan);
  }
  return hipGetLastError();
}

hipError_t launch_fill_i32(int* p, int value, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, wide_grid((n + 255) / 256), dim3(256), 0, s, p, value, n);
  return hipGetLastError();
}

hipError_t launch_clear_unpaired(const FrameDev& f, const int* counts, int m1, float* out, hipStream_t s) {
  const int64_t HW = int64_t(f.W) * f.H, chunks = (HW + CLEAR_THREADS - 1) / CLEAR_THREADS;
  hipLaunchKernelGGL(k_clear_unpaired, wide_grid(chunks * f.n_slots), dim3(CLEAR_THREADS), 0, s, counts, f.n_slots, m1,
                     f.W, HW, f.tw_log2, f.tiles_x, chunks, out);
  return hipGetLastError();
}

hipError_t launch_incidence_count(const int4* tv, int64_t n_tets, int* counts, hipStream_t s) {
  hipLaunchKernelGGL(k_inc_count, dim3(grid1(n_tets, 256)), dim3(256), 0, s, tv, n_tets, counts);
  return hipGetLastError();
}

hipError_t launch_incidence_fill(const int4* tv, int64_t n_tets, const int* offsets, int* cursors, int* inc,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_inc_fill, dim3(grid1(n_tets, 256)), dim3(256), 0, s, tv, n_tets, offsets, cursors, inc);
  return hipGetLastError();
}

hipError_t launch_adjacency(const int4* tv, int64_t n_tets, const int* offsets, const int* inc, int* nbr,
                            int* err, hipStream_t s) {
  hipLaunchKernelGGL(k_adjacency, dim3(grid1(4 * n_tets, 256)), dim3(256), 0, s, tv, n_tets, offsets, inc, nbr,
                     err);
  return hipGetLastError();
}

}  // namespace apc

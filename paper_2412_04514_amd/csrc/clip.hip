// Cell clipping with the security-radius certificate (paper, Summary section:
// each cell starts as a bounding box that is cut, one neighbour at a time, by
// the bisector plane between the generator and that neighbour, and a
// security-radius condition proves the result complete; the radius lemma is
// the one of Ray et al. 2018, cited by the paper).
//
// MI355X design
//  * A group of L lanes owns one cell; a 64-lane wave (= one workgroup) holds
//    64/L cells.  Lane j of a group handles vertex slots t = j, j+L, ...
//  * Three kernels: the list kernel (8 lanes per cell) clips every cell by its
//    list; cells that the list does not certify go on, with the polyhedron it
//    left, in the stream kernel (16 lanes per cell), and cells that outgrow both
//    go to the large-capacity kernel (32 lanes).  The stream kernel does both
//    phases where there is no list, or no place for a cell's state.  Vector
//    instructions bind the first (VALU busy 84%), loads, enumeration and the
//    unlike lengths of its four cells the second (57%).
//  * The polyhedron is kept in dual form in LDS: a list of clipping planes
//    (box walls + bisectors, at most PMAX alive at once, slots recycled) and a
//    list of triangles, one per vertex, each naming its three planes in
//    counter-clockwise order seen from outside.  Vertex positions are cached
//    next to the triangles, in seed-relative coordinates.
//  * Clipping by plane m: every lane tests its vertices (n.v > c means
//    outside), a ballot tells the group whether anything is cut.  For a cut,
//    the removed triangles are listed one per lane, and their directed dual
//    edges are marked in a per-cell bit matrix; an edge whose twin is unmarked
//    lies on the boundary of the removed region and becomes a new triangle
//    (a, b, m).  New vertices are solved from their three planes (Cramer), so
//    no error accumulates from earlier vertices.  A plane with removed
//    triangles and no boundary edge has lost its face; the radius R^2 is
//    rebuilt with a group reduction.
//  * Certificate: before plane m, the cell is final when d_m^2 > 4 R^2; after
//    the list, when d_k^2 > 4 R^2 or the list holds every other point.
//  * Volume: sum over vertices of corner terms det(F_f, v, e_fh - e_fg) / 6,
//    with F_f the foot of the seed on face f and e_fg the point of line f^g
//    nearest to the seed (a fan of each face from its foot, split at the edge
//    anchors), accumulated in double.
//  * Optional per-face outputs, in double from double vertices: the area of
//    each neighbour's face (the same corner terms, per face) and the cell
//    centroid (each corner term split into two signed tetrahedra from the
//    seed, weighted by their corner means).
//  * F32_RECHECK: tests and radii in float; a plane-side test whose margin is
//    below eps of its scale, and a certificate comparison with
//    |d^2 - 4 R^2| <= eps d^2, are redone in double from the exact inputs.
#include "internal.h"
#include "device_common.h"

#include <cfloat>

namespace votess {
namespace {

// A triangle's three plane slots in one word: 5 bits each in 16 bits where 32
// planes are enough, else 8 bits each.
template <int PMAX>
struct TriCode {
  using T = typename std::conditional<(PMAX <= 32), unsigned short, unsigned>::type;
  static constexpr int kShift = PMAX <= 32 ? 5 : 8;
  static constexpr unsigned kMask = (1u << kShift) - 1u;
  static constexpr unsigned kEmpty = PMAX <= 32 ? 0xFFFFu : 0xFFFFFFFFu;
  __device__ static unsigned make(unsigned a, unsigned b, unsigned c) { return a | (b << kShift) | (c << 2 * kShift); }
  __device__ static int a(unsigned u) { return (int)(u & kMask); }
  __device__ static int b(unsigned u) { return (int)((u >> kShift) & kMask); }
  __device__ static int c(unsigned u) { return (int)((u >> 2 * kShift) & kMask); }
};
constexpr int ST_RUN = -1;

struct ClipArgs {
  const void* rec;
  int n;
  double lo0, lo1, lo2, hi0, hi1, hi2;
  const int* cells;
  int nc;
  const int* knn;
  int k;
  int kstride;    // entries per list row
  int knn_by_id;  // list row of a cell: its sorted id (else its position in cells)
  double eps;
  double dmargin;  // applied to d^2 in certificate tests (k-lists built in float)
  int max_nbr, max_vert, out_by_id;
  uint8_t* status;
  int* nbr_count;
  int* nbr;
  double* volume;
  int* kneeded;
  int* vcount;
  double* verts;
  int* vplanes;
  double* area;      // [rows, max_nbr] next to nbr (nullable)
  double* centroid;  // [rows, 3] (nullable)
  double* r2out;     // [rows] (nullable): R^2 of the certified cell (an upper bound on the float path)
  unsigned long long* counters;
  int level[kLevels];
  // passing cells on from the list kernel to a second launch (see k_clip):
  int rest;  // 1: only the cells that the list kernel left
  int per;   // cells per wave: 64 / L, or fewer
  int mark;  // statuses of cells that the list kernel leaves, as a bit mask
  int save;  // 1 (list kernel): uncertified cells leave their state in nbr
  // stream phase (cells the list did not certify keep clipping by grid rings)
  int stream;
  const int* cell_start;
  GridDev grid;
  SubGrid sub;  // sub-grids of dense cells (info null: none)
};

template <typename R>
struct V3 {
  R x, y, z;
};

template <typename R>
__device__ __forceinline__ V3<R> cross(const V3<R>& a, const V3<R>& b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename R>
__device__ __forceinline__ R dot(const V3<R>& a, const V3<R>& b) {
  return a.x * b.x + a.y * b.y + a.z * b.z;
}

// Vertex of planes a, b, c: solve [a; b; c] x = [ca, cb, cc].  Which products
// are fused, and which of a sum's first two terms is rounded first, is written
// out rather than left to the compiler, whose choice moves with the code around
// it: the kernels of a clip and the state passed between them must agree on
// every bit of a vertex, and so must one build with the next.  (FIRST: the first
// term of det, not of y and z, as the float clip's rechecks have it; the double
// clip has them the other way round.)
template <bool FIRST>
__device__ __forceinline__ V3<double> solve3(const V3<double>& a, double ca, const V3<double>& b, double cb,
                                             const V3<double>& c, double cc) {
#pragma clang fp contract(off)
  auto fma = [](double x, double y, double z) { return __builtin_fma(x, y, z); };
  auto cross_ = [&](const V3<double>& p, const V3<double>& q) -> V3<double> {
    return {fma(p.y, q.z, -(p.z * q.y)), fma(p.z, q.x, -(p.x * q.z)), fma(p.x, q.y, -(p.y * q.x))};
  };
  // p q + r s with r s (last) or p q (first) rounded by itself
  auto sum2 = [&](bool first, double p, double q, double r, double s) {
    return first ? fma(r, s, p * q) : fma(p, q, r * s);
  };
  const V3<double> bc = cross_(b, c), cx = cross_(c, a), ab = cross_(a, b);
  const double inv = 1.0 / fma(a.z, bc.z, sum2(FIRST, a.x, bc.x, a.y, bc.y));
  return {fma(cc, ab.x, sum2(false, ca, bc.x, cb, cx.x)) * inv, fma(cc, ab.y, sum2(!FIRST, ca, bc.y, cb, cx.y)) * inv,
          fma(cc, ab.z, sum2(!FIRST, ca, bc.z, cb, cx.z)) * inv};
}

// c - n.v as if in twice the working precision: each product split exactly
// by an FMA, each sum by an error-free two-sum, the error terms added last.
// The residual of a vertex of nearly singular planes survives cancellation.
__device__ __forceinline__ double residual2(const V3<double>& n, double c, const V3<double>& v) {
#pragma clang fp contract(off)
  double s = c, err = 0.0;
  const double a[3] = {n.x, n.y, n.z}, b[3] = {v.x, v.y, v.z};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double p = a[i] * b[i];
    const double ep = fma(a[i], b[i], -p);  // a b = p + ep exactly
    const double t = s - p;                 // s - p = t + es exactly
    const double z = t - s;
    const double es = (s - (t - z)) + (-p - z);
    s = t;
    err += es - ep;
  }
  return s + err;
}

// The same residual for a bisector plane (n, |n|^2 / 2) without rounding its
// offset: c - n.v = sum_i n_i (n_i / 2 - v_i), each difference split by a
// two-sum, each product by an FMA.  The double offset |n|^2 / 2 is rounded by
// u c, which a vertex of nearly parallel planes amplifies by its
// conditioning; this residual has no such term (n itself is exact for float
// inputs).
__device__ __forceinline__ double residual_bis(const V3<double>& n, const V3<double>& v) {
#pragma clang fp contract(off)
  double s = 0.0, err = 0.0;
  const double a[3] = {n.x, n.y, n.z}, b[3] = {v.x, v.y, v.z};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double h = 0.5 * a[i];  // exact
    const double d = h - b[i];    // h - b = d + ed exactly
    const double z0 = d - h;
    const double ed = (h - (d - z0)) + (-b[i] - z0);
    const double p = a[i] * d;
    const double ep = fma(a[i], d, -p);  // a d = p + ep exactly
    const double t = s + p;              // s + p = t + es exactly
    const double z = t - s;
    const double es = (s - (t - z)) + (p - z);
    s = t;
    err += es + ep + a[i] * ed;
  }
  return s + err;
}

// Vertex of three planes, refined once against its accurate residual (for
// the planes flagged as bisectors, with their offsets taken exactly): a few
// ulps of |v| unless the normals are singular to within ~u.
__device__ __forceinline__ V3<double> solve3_refined(const V3<double>& na, double ca, bool ba, const V3<double>& nb,
                                                     double cb, bool bb, const V3<double>& nc, double cc, bool bc_) {
  const V3<double> bc = cross(nb, nc), ca_ = cross(nc, na), ab = cross(na, nb);
  const double inv = 1.0 / dot(na, bc);
  auto apply = [&](double x, double y, double z) -> V3<double> {
    return {(x * bc.x + y * ca_.x + z * ab.x) * inv, (x * bc.y + y * ca_.y + z * ab.y) * inv,
            (x * bc.z + y * ca_.z + z * ab.z) * inv};
  };
  const V3<double> v = apply(ca, cb, cc);
  const V3<double> d = apply(ba ? residual_bis(na, v) : residual2(na, ca, v), bb ? residual_bis(nb, v) : residual2(nb, cb, v),
                             bc_ ? residual_bis(nc, v) : residual2(nc, cc, v));
  return {v.x + d.x, v.y + d.y, v.z + d.z};
}

// Float vertex of three planes with a first-order forward error bound (max
// norm): rounding of the cross products, the sums, the division and of the
// plane data (normals may be off by an ulp, offsets by two).  What is fused is
// written out, as in solve3.
__device__ __forceinline__ V3<float> solve3_err(const V3<float>& a, float ca, const V3<float>& b, float cb,
                                                const V3<float>& c, float cc, float& err) {
#pragma clang fp contract(off)
  auto fma = [](float x, float y, float z) { return __builtin_fmaf(x, y, z); };
  const float b1 = b.z * c.y, b2 = b.x * c.z, b3 = b.y * c.x;
  const V3<float> bc = {fma(b.y, c.z, -b1), fma(b.z, c.x, -b2), fma(b.x, c.y, -b3)};
  const float c1 = c.z * a.y, c2 = c.x * a.z, c3 = c.y * a.x;
  const V3<float> cx = {fma(c.y, a.z, -c1), fma(c.z, a.x, -c2), fma(c.x, a.y, -c3)};
  const float a1 = a.z * b.y, a2 = a.x * b.z, a3 = a.y * b.x;
  const V3<float> ab = {fma(a.y, b.z, -a1), fma(a.z, b.x, -a2), fma(a.x, b.y, -a3)};
  const V3<float> pbc = {fabsf(b.y * c.z) + fabsf(b1), fabsf(b.z * c.x) + fabsf(b2), fabsf(b.x * c.y) + fabsf(b3)};
  const V3<float> pca = {fabsf(c.y * a.z) + fabsf(c1), fabsf(c.z * a.x) + fabsf(c2), fabsf(c.x * a.y) + fabsf(c3)};
  const V3<float> pab = {fabsf(a.y * b.z) + fabsf(a1), fabsf(a.z * b.x) + fabsf(a2), fabsf(a.x * b.y) + fabsf(a3)};
  const float det = fma(a.z, bc.z, fma(a.y, bc.y, a.x * bc.x));
  const float inv = 1.0f / det;
  const V3<float> v = {fma(cc, ab.x, fma(cb, cx.x, ca * bc.x)) * inv, fma(cc, ab.y, fma(cb, cx.y, ca * bc.y)) * inv,
                       fma(cc, ab.z, fma(ca, bc.z, cb * cx.z)) * inv};
  const float u8 = 8.0f * (0.5f * FLT_EPSILON);
  const float dD = u8 * fma(fabsf(a.z), pbc.z, fma(fabsf(a.y), pbc.y, fabsf(a.x) * pbc.x));
  const float ka = fabsf(ca), kb = fabsf(cb), kc = fabsf(cc);
  const float ai = fabsf(inv);
  const float sx = fma(kc, pab.x, fma(kb, pca.x, ka * pbc.x)), sy = fma(kc, pab.y, fma(kb, pca.y, ka * pbc.y)),
              sz = fma(kc, pab.z, fma(ka, pbc.z, kb * pca.z));
  const float ex = fma(FLT_EPSILON, fabsf(v.x), fma(u8, sx, fabsf(v.x) * dD) * ai);
  const float ey = fma(FLT_EPSILON, fabsf(v.y), fma(u8, sy, fabsf(v.y) * dD) * ai);
  const float ez = fma(FLT_EPSILON, fabsf(v.z), fma(u8, sz, fabsf(v.z) * dD) * ai);
  err = fmaxf(ex, fmaxf(ey, ez));
  return v;
}

template <typename M>
__device__ __forceinline__ M bitm(int i) {
  return M(1) << i;
}

// Lane moves inside a row of 16 lanes by DPP, which stays in the vector ALU
// (controls: quad_perm [1,0,3,2] = 0xB1 takes lane ^ 1, [2,3,0,1] = 0x4E
// lane ^ 2; row_shr:n = 0x110 + n takes lane - n; row_mirror = 0x140 takes lane 15 - i, row_half_mirror = 0x141
// lane 7 - i within each eight).  Moves across rows use the LDS permute.
template <int CTRL>
__device__ __forceinline__ unsigned dpp_mov(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// the word of lane - n (n = 1, 2, 4, 8; lanes below n of the row receive 0)
__device__ __forceinline__ unsigned up_word(unsigned v, int n) {
  switch (n) {
    case 1: return dpp_mov<0x111>(v);
    case 2: return dpp_mov<0x112>(v);
    case 4: return dpp_mov<0x114>(v);
    default: return dpp_mov<0x118>(v);
  }
}
// one step of a reduction over a group of w lanes: the value of the lane that
// the step of width o = 1, 2, 4, 8, 16 combines with this one.  After the
// steps before it, all lanes of a block of o hold the same value, so any lane
// of the neighbouring block will do, and one DPP move finds one (within a row
// of 16 lanes: quad_perm, row_half_mirror, row_mirror).  Every lane of the
// group is active.
__device__ __forceinline__ unsigned step_word(unsigned v, int o) {
  switch (o) {
    case 1: return dpp_mov<0xB1>(v);
    case 2: return dpp_mov<0x4E>(v);
    case 4: return dpp_mov<0x141>(v);
    case 8: return dpp_mov<0x140>(v);
    default: return (unsigned)__shfl_xor((int)v, o, 64);
  }
}
template <typename T>
__device__ __forceinline__ T red_step(T v, int o) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two words");
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, step_word(__builtin_bit_cast(unsigned, v), o));
  } else {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned long long r =
        ((unsigned long long)step_word((unsigned)(u >> 32), o) << 32) | step_word((unsigned)u, o);
    return __builtin_bit_cast(T, r);
  }
}

// value of wave lane src
__device__ __forceinline__ float shfl_t(float v, int src) { return __shfl(v, src, 64); }
__device__ __forceinline__ double shfl_t(double v, int src) { return __shfl(v, src, 64); }

// FP64 plane of a cell (generator p): the bisector with point `id` (>= 0) or
// box wall -id-1 (x-, x+, y-, y+, z-, z+); n . x <= c relative to p.  All
// arguments are values, so that no selection below goes through memory.
template <typename Rec4>
__device__ __forceinline__ void plane64_of(int id, const Rec4* rec, double px, double py, double pz, double lo0,
                                           double lo1, double lo2, double hi0, double hi1, double hi2, V3<double>& n,
                                           double& c) {
  if (id >= 0) {
    const Rec4 q = rec[id];
    n = {(double)q.x - px, (double)q.y - py, (double)q.z - pz};
    c = 0.5 * dot(n, n);
  } else {
    const int w = -id - 1, ax = w >> 1;
    const bool hi = w & 1;
    const double lo_a = ax == 0 ? lo0 : (ax == 1 ? lo1 : lo2);
    const double hi_a = ax == 0 ? hi0 : (ax == 1 ? hi1 : hi2);
    const double p_a = ax == 0 ? px : (ax == 1 ? py : pz);
    const double sgn = hi ? 1.0 : -1.0;
    n = {ax == 0 ? sgn : 0.0, ax == 1 ? sgn : 0.0, ax == 2 ? sgn : 0.0};
    c = hi ? hi_a - p_a : p_a - lo_a;
  }
}

// State of a cell between the list kernel and the stream kernel, in the
// cell's own neighbour row: the plane ids by slot (32 words; n and c follow
// from the id), the alive mask, the number of triangles, and the triangles as
// three 5-bit plane slots in 16 bits, in the order (a, b, last applied), from
// which the stream kernel solves the same vertices again, bit for bit.
// Mark in a status: the list kernel left the cell to the second launch.
constexpr uint8_t kLeft = 0x80;
constexpr int kListLanes = 8, kListVert = 48;  // lanes per cell and vertex slots of the list kernel
constexpr int kStateAlive = 32, kStateCount = 33, kStateTri = 34, kStateWords = kStateTri + kListVert / 2;

// A launch over nc cells, `per` to a wave (= block), in units of `per` cells or,
// with `rest`, of 64 that 64 / per waves share.  Blocks are dealt round-robin over
// the eight XCDs.  Each XCD takes every eighth of up to 8 kStretches contiguous
// stretches of units: its L2 then holds a stretch's neighbours, and dense and
// sparse regions fall to all XCDs alike.  Within a stretch come the first waves
// of all units, then their second ones, ...: the waves that find nothing are the
// later ones of a unit, and in unit order they fell to the same shader engines
// again and again.  Clip times with one stretch per XCD in unit order, with one
// in wave order, with 64 and with 256: 16M clustered points 199, 186, 189 and
// 188 ms; 3M in double 50.4, 48.4, 48.6 and 47.0; 1.2M filament points with
// faces 43.2, 41.3, 38.1 and 37.5; 1M uniform ones 6.32, 5.73, 5.73 and 5.76.
constexpr int kStretches = 256;
struct ClipGrid {
  int units, waves, len, stretches;  // units, waves of each; units of a stretch, stretches per XCD
  __host__ __device__ __forceinline__ ClipGrid(int nc, int per, int rest) {
    units = (int)(((long long)nc + (rest ? 64 : per) - 1) / (rest ? 64 : per));
    waves = rest ? 64 / per : 1;
    const int eighth = (int)(((long long)units + 7) / 8);
    stretches = eighth < kStretches ? eighth : kStretches;
    len = (eighth + stretches - 1) / stretches;
  }
  __host__ __device__ __forceinline__ unsigned blocks() const {
    return 8u * (unsigned)stretches * (unsigned)len * (unsigned)waves;
  }
  __host__ __device__ __forceinline__ void find(unsigned b, int& unit, int& wave) const {
    const int i = (int)(b >> 3), stretch = i / (len * waves), at = i - stretch * len * waves;
    wave = at / len;
    unit = (stretch * 8 + (int)(b & 7u)) * len + (at - wave * len);
  }
};

// Clips 64 / L cells, one per group of L lanes: cell t_idx of the launch (no
// cell when !have), from its box or, when `resume`, from the state that the
// list kernel left.
template <typename P, typename R, int L, int TMAX, int PMAX, bool RECHECK, bool STREAM>
__device__ __forceinline__ void clip_group(const ClipArgs& a, long long t_idx, bool have, bool resume) {
  using Rec4 = typename Rec<P>::type;
  using M = typename std::conditional<(PMAX <= 32), unsigned, unsigned long long>::type;
  constexpr int G = 64 / L;
  constexpr int S = TMAX / L;
  constexpr int TP = TMAX + 1;
  constexpr M PFULL = (PMAX == 8 * (int)sizeof(M)) ? ~M(0) : ((M(1) << PMAX) - 1);
  static_assert(S <= 32, "slot mask is 32 bits");
  static_assert(TMAX % L == 0 && TMAX % 4 == 0, "the slots are taken L at a time, or 4");
  static_assert(L <= 32, "a group's ballot is taken from one word");
  static_assert(RECHECK == (sizeof(R) == 4), "the float clip rechecks, the double one does not");
  static_assert(TMAX <= 256, "vertex slots are numbered in one byte");

  // Vertices: float ones as (x, y, z, forward error bound), so that a vertex
  // is one 16-byte read; double ones by coordinate.  An empty slot holds
  // zeros: its plane tests read -c < 0, never cut, without a look at tri.
  constexpr int V4 = RECHECK ? G * TP : 1, VD = RECHECK ? 1 : G * TP;
  __shared__ float4 vtx[V4];
  __shared__ R vx[VD], vy[VD], vz[VD];
  using TC = TriCode<PMAX>;
  constexpr unsigned kEmpty = TC::kEmpty;
  __shared__ typename TC::T tri[G * TP];
  // planes: a bisector's normal and the id of its point, float ones as 16
  // bytes; with float points a double clip keeps the point itself (exact, and
  // half the size).  The offset follows from the normal.  Of a wall only the
  // id is read.
  constexpr bool kPoint = sizeof(P) == 4 && sizeof(R) == 8;
  constexpr int P4 = sizeof(P) == 4 ? G * PMAX : 1, PD = sizeof(P) == 4 ? 1 : G * PMAX;
  __shared__ float4 pn4[P4];
  __shared__ double pnx[PD], pny[PD], pnz[PD];
  __shared__ int pidd[PD];
  __shared__ M omask[G * PMAX];
  __shared__ unsigned short snew[G * (PMAX + 1)];
  // free vertex slots below H, as a stack; a cut pushes the slots it removes,
  // so that its top then lists the removed triangles
  __shared__ unsigned char fstk[G * TP];
  // stream phase: the vertices in reach and their balls, and those of them
  // whose ball meets the dense cell being scanned (see below)
  constexpr int kReach = TMAX <= 64 ? 48 : TMAX;
  constexpr int RVN = STREAM ? G * kReach : 1;
  // (float: centre and radius, one 16-byte read; double: the vertex slot and the
  // radius, half the LDS of a copy: 3M clustered points 64.2 and 70.4 ms.  The few
  // waves of the large kernel wait for each read and have LDS to spare: copies, 10k
  // clustered points in double 2.80 and 2.59 ms.)
  struct alignas(16) Ball {
    R x, y, z, r;
  };
  // Tests against them read four at a time, so that their latency is met once: 200k
  // clustered points, double clip, 7.36 -> 6.95 ms, 300k in float without lists
  // 8.59 -> 7.95; by two 7.17 and 8.19, by eight spills.
  constexpr int kAhead = 4;
  constexpr bool kCopies = RECHECK || TMAX > 64;
  constexpr int RVF = STREAM && kCopies ? G * kReach : 1, RVD = STREAM && !kCopies ? G * kReach : 1;
  __shared__ Ball reachv[RVF];
  __shared__ R reachr[RVD];
  __shared__ unsigned char reachs[RVD];
  __shared__ unsigned char relD[RVN];
  // stream phase: sub-cell widths of the dense cell being scanned, per group
  constexpr int DG = STREAM ? G * 3 : 1;
  __shared__ double dgeo[DG];
  // stream phase: the flower box in coordinates, per group (read only when a
  // dense cell is entered, so it need not occupy registers)
  constexpr int FWG = STREAM ? G * 6 : 1;
  __shared__ double fwbox[FWG];
  // stream phase: listed parts of the ring, and point ranges of up to L
  // sub-rows of the dense cell being scanned (offsets into the cell), per group
  constexpr int SRL = STREAM ? G * L : 1;
  __shared__ int2 rowlist[SRL], srl[SRL];
  // stream phase: the group's enumeration state (grid ring, x-run, dense
  // sub-block, flower box in cells).  Every value is the same for all lanes
  // of a group; held here rather than in registers, which the rest of the
  // kernel needs.
  struct Enum {
    int fb0, fb1, fb2, fb3, fb4, fb5;
    int rr, pq, np, zlo, ylo, nyr, rln, rlp;
    int rx, rx1, rrow, yy, zz;
    int dm, dm0, dm1, dm2, dbase, dsx0, dsx1, dsy0, dsy1, dsz0, dsz1, dsto;
    int dq1, dq2, kyn, kzn, dq, dqn, srn, srp;
  };
  __shared__ Enum senum[STREAM ? G : 1];

  const Rec4* rec = (const Rec4*)a.rec;
  const int lane = threadIdx.x;
  const int g = lane / L, j = lane % L;
  const int gb = g * L;
  const int vb = g * TP, pb = g * PMAX, sb = g * (PMAX + 1);
  const int sid = have ? (a.cells ? a.cells[t_idx] : (int)t_idx) : 0;
  const int row = a.out_by_id ? sid : (int)t_idx;
  const Rec4 pr = rec[sid];
  const double p64x = pr.x, p64y = pr.y, p64z = pr.z;
  const R px = (R)pr.x, py = (R)pr.y, pz = (R)pr.z;

  // the group's bits of a ballot
  auto gballot = [&](bool v) -> unsigned {
    const unsigned long long b = __ballot(v);
    const unsigned w = lane >= 32 ? (unsigned)(b >> 32) : (unsigned)b;
    if constexpr (L == 32) return w;
    return __builtin_amdgcn_ubfe(w, gb & 31, L);
  };
  const unsigned below = (1u << j) - 1u;  // the group's lanes before this one
  auto group_any = [&](bool v) -> bool { return gballot(v) != 0u; };
  auto gor = [&](M v) -> M {
#pragma unroll
    for (int o = 1; o < L; o <<= 1) v |= red_step(v, o);
    return v;
  };
  auto gmax = [&](R v) -> R {
#pragma unroll
    for (int o = 1; o < L; o <<= 1) v = fmax(v, red_step(v, o));
    return v;
  };
  auto gsumd = [&](double v) -> double {
#pragma unroll
    for (int o = 1; o < L; o <<= 1) v += red_step(v, o);
    return v;
  };
  // exclusive prefix sum over the group's lanes, and the total
  auto gexcl = [&](int v, int& tot) -> int {
    int x = v;
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
      const int y = L <= 16 ? (int)up_word((unsigned)x, o) : __shfl_up(x, o, L);
      if (j >= o) x += y;
    }
    tot = v;
#pragma unroll
    for (int o = 1; o < L; o <<= 1) tot += red_step(tot, o);
    return x - v;
  };

  // the id of the plane in slot f: a point's, or -1 - wall
  auto pid = [&](int f) -> int {
    if constexpr (sizeof(P) == 4) return __float_as_int(pn4[pb + f].w);
    else return pidd[pb + f];
  };
  // FP64 plane of slot f, from the exact inputs (used by the recheck).
  const double blo0 = a.lo0, blo1 = a.lo1, blo2 = a.lo2, bhi0 = a.hi0, bhi1 = a.hi1, bhi2 = a.hi2;
  auto plane64 = [&](int f, V3<double>& n, double& c) {
    plane64_of(pid(f), rec, p64x, p64y, p64z, blo0, blo1, blo2, bhi0, bhi1, bhi2, n, c);
  };
  auto vertex64 = [&](unsigned u) -> V3<double> {
    V3<double> na, nb, nc;
    double ca, cb, cc;
    plane64(TC::a(u), na, ca);
    plane64(TC::b(u), nb, cb);
    plane64(TC::c(u), nc, cc);
    return solve3<RECHECK>(na, ca, nb, cb, nc, cc);
  };

  auto vget = [&](int t) -> V3<R> {
    if constexpr (RECHECK) {
      const float4 v = vtx[vb + t];
      return {v.x, v.y, v.z};
    } else {
      return {vx[vb + t], vy[vb + t], vz[vb + t]};
    }
  };
  auto vget_err = [&](int t, float& e) -> V3<R> {
    if constexpr (RECHECK) {
      const float4 v = vtx[vb + t];
      e = v.w;
      return {v.x, v.y, v.z};
    } else {
      e = 0.0f;
      return {vx[vb + t], vy[vb + t], vz[vb + t]};
    }
  };
  auto vput = [&](int t, R x, R y, R z, float e) {
    if constexpr (RECHECK) {
      vtx[vb + t] = make_float4(x, y, z, e);
    } else {
      vx[vb + t] = x;
      vy[vb + t] = y;
      vz[vb + t] = z;
    }
  };
  auto pget = [&](int f, V3<R>& n, R& c) {
    int id;
    if constexpr (sizeof(P) == 4) {
      const float4 q = pn4[pb + f];
      id = __float_as_int(q.w);
      if constexpr (kPoint) n = {(R)q.x - px, (R)q.y - py, (R)q.z - pz};
      else n = {(R)q.x, (R)q.y, (R)q.z};
    } else {
      n = {(R)pnx[pb + f], (R)pny[pb + f], (R)pnz[pb + f]};
      id = pidd[pb + f];
    }
    c = R(0.5) * dist2_nc(n.x, n.y, n.z);
    if (id < 0) {
      V3<double> w;
      double cw;
      plane64_of(id, rec, p64x, p64y, p64z, blo0, blo1, blo2, bhi0, bhi1, bhi2, w, cw);
      n = {(R)w.x, (R)w.y, (R)w.z};
      c = (R)cw;
    }
  };
  // the bisector with point id, whose normal is (nx, ny, nz) and, where points
  // are kept, its position (qx, qy, qz)
  auto pput = [&](int f, R nx, R ny, R nz, float qx, float qy, float qz, int id) {
    if constexpr (sizeof(P) == 4) {
      if constexpr (kPoint) pn4[pb + f] = make_float4(qx, qy, qz, __int_as_float(id));
      else pn4[pb + f] = make_float4((float)nx, (float)ny, (float)nz, __int_as_float(id));
    } else {
      pnx[pb + f] = nx;
      pny[pb + f] = ny;
      pnz[pb + f] = nz;
      pidd[pb + f] = id;
    }
  };

  // ---- initial cell: the box, in seed-relative coordinates
  for (int t = j; t < TMAX; t += L) {
    tri[vb + t] = (typename TC::T)kEmpty;
    vput(t, R(0), R(0), R(0), 0.0f);
  }
  for (int f = j; f < PMAX; f += L) omask[pb + f] = 0;
  const R lx = (R)(a.lo0 - p64x), hx = (R)(a.hi0 - p64x);
  const R ly = (R)(a.lo1 - p64y), hy = (R)(a.hi1 - p64y);
  const R lz = (R)(a.lo2 - p64z), hz = (R)(a.hi2 - p64z);
  for (int v = j; v < 8; v += L) {
    const int bx = v & 1, by = (v >> 1) & 1, bz = (v >> 2) & 1;
    const R X0 = bx ? hx : lx, Y0 = by ? hy : ly, Z0 = bz ? hz : lz;
    const unsigned X = bx, Y = 2 + by, Z = 4 + bz;
    // (X, Y, Z) is counter-clockwise seen from outside iff an odd number of
    // the three coordinates are on the high side
    tri[vb + v] = (typename TC::T)(((bx + by + bz) & 1) ? TC::make(X, Y, Z) : TC::make(X, Z, Y));
    vput(v, X0, Y0, Z0,
         RECHECK ? FLT_EPSILON * (float)fmax(fabs((double)X0), fmax(fabs((double)Y0), fabs((double)Z0))) : 0.0f);
  }
  for (int f = j; f < 6; f += L) pput(f, R(0), R(0), R(0), 0.0f, 0.0f, 0.0f, -(f + 1));
  int st = have ? ST_RUN : VOTESS_CELL_CERTIFIED;
  int H = 8;   // slots in use lie below H
  int nfr = 0;  // free slots below H (fstk)
  M alive = M(0x3F);
  R R2 = fmax(lx * lx, hx * hx) + fmax(ly * ly, hy * hy) + fmax(lz * lz, hz * hz);
  // float path: R2 is the largest |v|^2 of the float vertices.  The true R^2
  // lies between bounds made from each vertex's forward error bound err,
  // R2lo <= R^2 <= R2hi, and a radius test is rechecked only between them.
  // By how vertices are made err <= max(16 eps, FLT_EPSILON) |v|, so both
  // bounds lie within a relative kap of R2: a distance d^2 of at most rlo is
  // certainly no certificate, one above rhi certainly is one, and only in
  // between (rarely) are the bounds worked out.
  const float verrel = fmaxf(16.0f * (float)a.eps, FLT_EPSILON);
  const float kap = (3.5f + verrel) * verrel + 2.0f * (float)a.eps + 4e-6f;
  float R2up = 0.0f, rlo = 0.0f, rhi = 0.0f;
  auto set_radius = [&](R r2) {
    R2 = r2;
    if constexpr (RECHECK) {
      R2up = r2 * (1.0f + kap);
      rlo = 4.0f * r2 * (1.0f - kap);
      rhi = 4.0f * R2up;
    }
  };
  set_radius(R2);
  // |v| (1 + 1e-5) + 4 verr.  verr bounds each coordinate of the float
  // vertex, so the true ball's centre lies within verr per axis and its radius
  // within sqrt(3) verr: 4 verr > (1 + sqrt(3)) verr covers both; the relative
  // 1e-5 covers the rounding of this radius and of the box-ball tests, made in
  // the clip's precision.
  auto ball_rad = [&](R X, R Y, R Z, float e) -> R {
    if constexpr (sizeof(R) == 4) {
      return sqrtf(X * X + Y * Y + Z * Z) * (1.0f + 1e-5f) + 4.0f * e;
    } else {
      return sqrt(X * X + Y * Y + Z * Z) * (1.0 + 1e-5);
    }
  };
  bool streamed = false;  // the cell has entered the stream phase
  int kneed = 0;  // unresolved at plane m of the list: -1 - m
  int nrecheck = 0;
  __syncthreads();

  // Recheck of the security radius in double: R^2 from vertices solved in FP64.
  auto radius64 = [&](bool need) -> double {
    double r2 = 0.0;
    if (need) {
      for (int t = j; t < H; t += L) {
        const unsigned u = tri[vb + t];
        if (u == kEmpty) continue;
        const V3<double> v = vertex64(u);
        r2 = fmax(r2, dot(v, v));
      }
    }
#pragma unroll
    for (int o = 1; o < L; o <<= 1) r2 = fmax(r2, red_step(r2, o));
    return r2;
  };
  const double kDmargin = a.dmargin;
  // Vertex of planes A, B and the later one (n, c) in slot C.  A float vertex
  // comes with its error bound, and from double when that is too large.
  auto vertex = [&](int A, int B, int C, R nx, R ny, R nz, R c, float& ev, bool& redone) -> V3<R> {
    V3<R> na, nb_, v;
    R ca, cb;
    pget(A, na, ca);
    pget(B, nb_, cb);
    ev = 0.0f;
    redone = false;
    if constexpr (RECHECK) {
      v = solve3_err(na, ca, nb_, cb, {nx, ny, nz}, c, ev);
      const float vm = fmaxf(fabsf(v.x), fmaxf(fabsf(v.y), fabsf(v.z)));
      if (!(ev <= 16.0 * a.eps * vm)) {
        // ill-conditioned float vertex: solve it in double from the exact
        // planes and keep the rounded value (bound: one ulp)
        const V3<double> w = vertex64(TC::make(A, B, C));
        v = {(float)w.x, (float)w.y, (float)w.z};
        ev = FLT_EPSILON * (float)fmax(fabs(w.x), fmax(fabs(w.y), fabs(w.z)));
        redone = true;
      }
    } else {
      v = solve3<RECHECK>(na, ca, nb_, cb, {nx, ny, nz}, c);
    }
    return v;
  };
  if constexpr (STREAM) {
    if (resume) {
      const int* w = a.nbr + (size_t)row * a.max_nbr;
      H = w[kStateCount];
      alive = (M)(unsigned)w[kStateAlive];
      for (int f = j; f < 32; f += L) {
        const int id = w[f];
        if (!((alive >> f) & 1)) continue;
        const Rec4 q = rec[id >= 0 ? id : sid];
        pput(f, (R)q.x - px, (R)q.y - py, (R)q.z - pz, (float)q.x, (float)q.y, (float)q.z, id);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      const unsigned short* tr = (const unsigned short*)(w + kStateTri);
      R r2 = 0;
      for (int t = j; t < (H + L - 1) / L * L; t += L) {
        if (t < H) {
          const unsigned x = tr[t];
          const int A = TriCode<32>::a(x), B = TriCode<32>::b(x), C = TriCode<32>::c(x);
          V3<R> n, v;
          R c;
          float e;
          bool redone;
          pget(C, n, c);
          v = vertex(A, B, C, n.x, n.y, n.z, c, e, redone);
          if (pid(A) < 0 && pid(B) < 0 && pid(C) < 0) {
            e = FLT_EPSILON * (float)fmax(fabs((double)v.x), fmax(fabs((double)v.y), fabs((double)v.z)));  // a box corner
          }
          vput(t, v.x, v.y, v.z, e);
          tri[vb + t] = (typename TC::T)TC::make(A, B, C);
          r2 = fmax(r2, v.x * v.x + v.y * v.y + v.z * v.z);
        } else if (t < TMAX) {
          tri[vb + t] = (typename TC::T)kEmpty;
          vput(t, R(0), R(0), R(0), 0.0f);
        }
      }
      set_radius(gmax(r2));
      st = VOTESS_CELL_RADIUS;
    }
    __syncthreads();
  }
  // the float path's radius predicates by the bounds: bit 0 certain, bit 1
  // uncertain (else certainly not).  Called by whole groups.
  auto radius_bounds = [&](R dd2) -> int {
    float hi = 0.0f, lo = 0.0f;
    for (int t = j; t < H; t += L) {
      float e;
      const V3<R> v = vget_err(t, e);
      const float n2 = (float)(v.x * v.x + v.y * v.y + v.z * v.z), n1 = (float)(fabs(v.x) + fabs(v.y) + fabs(v.z));
      hi = fmaxf(hi, n2 + e * (2.0f * n1 + e));
      lo = fmaxf(lo, n2 - 2.0f * e * n1);
    }
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
      hi = fmaxf(hi, red_step(hi, o));
      lo = fmaxf(lo, red_step(lo, o));
    }
    hi *= 1.0f + 4.0f * FLT_EPSILON;
    lo *= 1.0f - 4.0f * FLT_EPSILON;
    if ((double)dd2 * kDmargin * (1.0 - a.eps) > 4.0 * (double)hi) return 1;
    return (double)dd2 * kDmargin * (1.0 + a.eps) > 4.0 * (double)lo ? 2 : 0;
  };

  // Bounds on the uncertainty window eps scale + |n|_1 err of a plane test of
  // the float clip: with |v| <= r, scale <= |n| r + c and |n|_1 <= sqrt(3) |n|;
  // by how vertices are made err <= max(16 eps, FLT_EPSILON) r.  A test outside
  // the bound is certain; one inside it works its own window out.
  // window(): for every vertex, window0(): less the |n|_1 err of the vertex.
  // (5e-7, in the candidates' test of the stream phase 2e-6, covers the roundings
  // of the float tests themselves: with an eps below 1e-6 they reach past the
  // rest.  |n| and |v| are rooted apart: the product of their squares leaves the
  // range of floats where the lengths are still in it.)
  const float wv = (float)a.eps + 1.7321f * verrel;
  auto window = [&](R d2, R c) -> R {
    if constexpr (RECHECK) {
      const float nv = __builtin_amdgcn_sqrtf(d2) * __builtin_amdgcn_sqrtf(R2up);
      return (((float)a.eps + 5e-7f) * c + (wv + 5e-7f) * nv) * (1.0f + 1e-4f);
    } else {
      return R(0);
    }
  };
  auto window0 = [&](R d2, R c) -> R {
    if constexpr (RECHECK) {
      const float nv = __builtin_amdgcn_sqrtf(d2) * __builtin_amdgcn_sqrtf(R2up);
      return (float)a.eps * (c + nv) * (1.0f + 1e-4f);
    } else {
      return R(0);
    }
  };

  // Tests plane (n, c) of candidate nb against every vertex and, if it cuts,
  // replaces the removed triangles; whether it did.  `m` is its place in the list
  // (-1: not of the list).  Called by every lane (wave-uniform).
  // Always inlined: as a call, its captures live in scratch memory.
  auto apply_plane = [&](bool run, R nx, R ny, R nz, R c, R d2, int nb, int m) __attribute__((always_inline)) -> bool {
    // ---- test the plane against every vertex
    unsigned out = 0;
    R least = R(3.0e38);  // the smallest margin of this lane's tests, less |n|_1 err
    const R nrm1 = (fabs(nx) + fabs(ny) + fabs(nz)) * R(1.0 + 1e-6);
    if (run) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (L * s < H) {
          float ev;
          const V3<R> v = vget_err(j + L * s, ev);
          const R sv = nx * v.x + ny * v.y + nz * v.z - c;
          if (sv > R(0)) out |= 1u << s;
          if constexpr (RECHECK) least = fmin(least, fabs(sv) - nrm1 * ev);
        }
      }
    }
    if constexpr (RECHECK) {
      const bool near = run && least <= window0(d2, c);
      if (__any(near)) {
        bool unresolved = false;
        for (int s = 0; near && L * s < H; ++s) {
          const int t = j + L * s;
          const unsigned u = tri[vb + t];
          if (u == kEmpty) continue;
          float ev;
          const V3<R> v = vget_err(t, ev);
          const R sv = nx * v.x + ny * v.y + nz * v.z - c;
          const R scale = fabs(nx * v.x) + fabs(ny * v.y) + fabs(nz * v.z) + c;
          const R nrm1 = fabs(nx) + fabs(ny) + fabs(nz);
          if (!(fabs(sv) <= (R)a.eps * scale + nrm1 * ev)) continue;
          const Rec4 q = rec[nb];
          const V3<double> n64 = {(double)q.x - p64x, (double)q.y - p64y, (double)q.z - p64z};
          const double c64 = 0.5 * dot(n64, n64);
          const V3<double> v64 = vertex64(u);
          const double s64 = dot(n64, v64) - c64;
          const double sc64 = fabs(n64.x * v64.x) + fabs(n64.y * v64.y) + fabs(n64.z * v64.z) + c64;
          if (fabs(s64) <= 1e-12 * sc64) unresolved = true;
          out = s64 > 0.0 ? out | (1u << s) : out & ~(1u << s);
          ++nrecheck;
        }
        if (group_any(unresolved) && run) {
          st = VOTESS_CELL_UNRESOLVED;
          if (m >= 0) kneed = -1 - m;
          run = false;
          out = 0;
        }
      }
    }
    const bool cut = run && group_any(out != 0u);
    if (!__any(cut)) return false;

    // ---- cut: new plane slot
    int ps = -1;
    bool doit = cut;
    if (doit) {
      const M fr = ~alive & PFULL;
      if (fr == M(0)) {
        st = VOTESS_CELL_CAPACITY;
        doit = false;
      } else {
        ps = (sizeof(M) == 4) ? (__ffs((unsigned)fr) - 1) : (__ffsll((unsigned long long)fr) - 1);
      }
    }
    if (doit && j == 0) {
      if constexpr (kPoint) {
        const Rec4 q = rec[nb];
        pput(ps, nx, ny, nz, (float)q.x, (float)q.y, (float)q.z, nb);
      } else {
        pput(ps, nx, ny, nz, 0.0f, 0.0f, 0.0f, nb);
      }
    }
    if (!doit) out = 0;
    // removed slots onto the free stack, which then lists them for the steps
    // below, one removed triangle per lane
    int rem = 0;
    {
      int w = nfr + gexcl(__popc(out), rem);
      for (unsigned left = out; left; left &= left - 1u) fstk[vb + w++] = (unsigned char)(j + L * (__ffs(left) - 1));
    }
    const bool many = __any(rem > L);
    __syncthreads();
    // mark the directed dual edges of removed triangles
    unsigned u = 0;
    for (int r0 = 0; __any(r0 < rem); r0 += L) {
      if (r0 + j < rem) {
        u = tri[vb + fstk[vb + nfr + r0 + j]];
        const int A = TC::a(u), B = TC::b(u), C = TC::c(u);
        atomicOr(&omask[pb + A], bitm<M>(B));
        atomicOr(&omask[pb + B], bitm<M>(C));
        atomicOr(&omask[pb + C], bitm<M>(A));
      }
    }
    __syncthreads();
    // boundary edges (twin not removed) become new triangles; a plane of a
    // removed triangle that starts no boundary edge has lost its face (the
    // boundary enters and leaves every face that is only cut)
    int btot = 0;
    M pr_ = 0, pk = 0;
    for (int r0 = 0; __any(r0 < rem); r0 += L) {
      const bool on = r0 + j < rem;
      bool e0 = false, e1 = false, e2 = false;
      int A = 0, B = 0, C = 0;
      if (on) {
        const int t = fstk[vb + nfr + r0 + j];
        if (many) u = tri[vb + t];
        A = TC::a(u), B = TC::b(u), C = TC::c(u);
        e0 = !((omask[pb + B] >> A) & 1);
        e1 = !((omask[pb + C] >> B) & 1);
        e2 = !((omask[pb + A] >> C) & 1);
        pr_ |= bitm<M>(A) | bitm<M>(B) | bitm<M>(C);
        pk |= (e0 ? bitm<M>(A) : M(0)) | (e1 ? bitm<M>(B) : M(0)) | (e2 ? bitm<M>(C) : M(0));
        tri[vb + t] = (typename TC::T)kEmpty;
        vput(t, R(0), R(0), R(0), 0.0f);
      }
      // edges are listed by lane; what is no edge, and (in an inconsistent
      // topology) an edge past the PMAX-th, goes to the spare entry PMAX
      const unsigned b0 = gballot(e0), b1 = gballot(e1), b2 = gballot(e2);
      const int o0 = btot + __popc(b0 & below) + __popc(b1 & below) + __popc(b2 & below), o1 = o0 + e0, o2 = o1 + e1;
      btot += __popc(b0) + __popc(b1) + __popc(b2);
      snew[sb + (e0 ? min(o0, PMAX) : PMAX)] = (unsigned short)(A | (B << 8));
      snew[sb + (e1 ? min(o1, PMAX) : PMAX)] = (unsigned short)(B | (C << 8));
      snew[sb + (e2 ? min(o2, PMAX) : PMAX)] = (unsigned short)(C | (A << 8));
    }
    __syncthreads();
    for (int f = j; f < PMAX; f += L) omask[pb + f] = 0;
    if (doit && (btot < 3 || btot > PMAX)) {  // inconsistent topology (rounding): give up on the cell
      st = VOTESS_CELL_UNRESOLVED;
      if (m >= 0) kneed = -1 - m;
      doit = false;
    }
    // new triangles (a, b, ps): into the freed slots, then past H
    const int avail = nfr + rem;
    const int hnew = H + max(0, btot - avail);
    if (doit && hnew > TMAX) {
      st = VOTESS_CELL_CAPACITY;
      doit = false;
    }
    for (int r = j; doit && r < btot; r += L) {
      const int t = r < avail ? (int)fstk[vb + avail - 1 - r] : H + r - avail;
      const unsigned e = snew[sb + r];
      const int A = e & 0xFF, B = (e >> 8) & 0xFF;
      float ev;
      bool redone;
      const V3<R> v = vertex(A, B, ps, nx, ny, nz, c, ev, redone);
      if (redone) ++nrecheck;
      vput(t, v.x, v.y, v.z, ev);
      tri[vb + t] = (typename TC::T)TC::make(A, B, ps);
    }
    __syncthreads();
    // R^2 over all slots (an empty one adds zero)
    R r2 = 0;
    if (doit) {
      H = hnew;
      nfr = max(0, avail - btot);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (L * s < H) {
          const V3<R> v = vget(j + L * s);
          r2 = fmax(r2, v.x * v.x + v.y * v.y + v.z * v.z);
        }
      }
    }
    r2 = gmax(r2);
    pr_ = gor(pr_);
    pk = gor(pk);
    if (doit) {
      alive = (alive & ~(pr_ & ~pk)) | bitm<M>(ps);
      set_radius(r2);
    }
    return doit;
  };

  // ---- list phase.  The list is taken in batches of L planes, one per lane.
  // A plane that cuts no vertex of the cell as it stands when its batch
  // begins never will (the cell only shrinks): one pass over the vertices
  // tests all L planes, and only those that may cut are applied, nearest
  // first.  Each group goes from one such plane to its next, whatever the
  // other groups of the wave do.  The certificate is checked in list order as
  // if plane by plane: before plane m, the cell is final when d_m^2 > 4 R^2,
  // R then being what the planes before m left.  The next batch's records and
  // the indices of the one after are loaded a batch ahead.  (Plane by plane
  // in step with the wave's other cells, every group waited at each plane that
  // cut any of them: the tessellation of 2^20 uniform points took 24.9 ms in
  // float, with batches 20.2 ms; 3M clustered points in double 145 and 131 ms.)
  const int* klist = a.knn + (size_t)(have ? (a.knn_by_id ? (long long)sid : t_idx) : 0) * a.kstride;
  {
    bool fin = !have || resume || a.k == 0;
    int mb = -L;     // list index of the batch's first plane
    int cur = L;     // first lane of the batch still to look at (L: none)
    unsigned pendb = 0, padb = 0;  // lanes whose plane may cut / lies past the list's end
    bool again = false;  // the plane of lane cur has just cut
    int id_c = -1, id_n = !fin && j < a.k ? klist[j] : -1, id_n2 = !fin && j + L < a.k ? klist[j + L] : -1;
    Rec4 q_n = rec[id_n >= 0 ? id_n : sid];
    R cx_ = 0, cy_ = 0, cz_ = 0, cd2 = 0;  // this lane's plane of the batch
    for (;;) {
      bool run = st == ST_RUN && !fin;
      if (!__any(run)) break;
      unsigned ev = 0, certb = 0, uncb = 0;
      while (run) {  // to the group's next plane that decides something
        if (cur < L) {
          const bool on = id_c >= 0;
          if constexpr (RECHECK) {
            certb = gballot(on && cd2 > rhi);
            uncb = 0u;
            if (gballot(on && cd2 > rlo && cd2 <= rhi) & (~0u << cur)) {
              const int p = radius_bounds(cd2);
              certb = gballot(on && p == 1);
              uncb = gballot(on && p == 2);
              // a plane that has cut is looked at again for the certificate
              // alone, and for a recheck only at the end of a list
              const int len = mb + cur + 1;
              if (again && len != a.k && len != a.level[0] && len != a.level[1] && len != a.level[2])
                uncb &= ~(1u << cur);
            }
          } else {
            certb = gballot(on && (R)(cd2 * (R)kDmargin) > R(4) * R2);
          }
          ev = (pendb | padb | certb | uncb) & (~0u << cur);
          if (ev) break;
        }
        mb += L;
        cur = 0;
        again = false;
        if (mb >= a.k) {
          fin = true;
          run = false;
          break;
        }
        const bool in = mb + j < a.k;
        id_c = in ? id_n : -1;
        const Rec4 q = q_n;
        id_n = id_n2;
        q_n = rec[id_n >= 0 ? id_n : sid];
        id_n2 = mb + 2 * L + j < a.k ? klist[mb + 2 * L + j] : -1;
        cx_ = (R)q.x - px;
        cy_ = (R)q.y - py;
        cz_ = (R)q.z - pz;
        cd2 = dist2_nc(cx_, cy_, cz_);
        const R c = R(0.5) * cd2;
        R far = -c;
        for (int t = 0; t < H; t += 4) {  // (slots from H to the next multiple of 4 are empty: zeros)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const V3<R> v = vget(t + i);
            far = fmax(far, cx_ * v.x + cy_ * v.y + cz_ * v.z);
          }
        }
        R w;
        if constexpr (RECHECK) w = window(cd2, c);
        else w = R(1e-12) * (c + sqrt(cd2 * R2));
        pendb = gballot(id_c >= 0 && !(far < c - w));
        padb = gballot(in && id_c < 0);
      }
      const int i = ev ? __ffs(ev) - 1 : 0, m = mb + i;
      const bool at_pad = (padb >> i) & 1u, at_cert = (certb >> i) & 1u;
      if (run && at_pad) {  // padded list: it holds every other point
        st = VOTESS_CELL_CERTIFIED;
        kneed = m;
        run = false;
      }
      if (run && at_cert) {
        st = VOTESS_CELL_CERTIFIED;
        kneed = m + 1;
        run = false;
      }
      const int nb = __shfl(id_c, gb + i, 64);
      if constexpr (RECHECK) {
        const bool need = run && ((uncb >> i) & 1u);
        if (__any(need)) {
          const double r64 = radius64(need);
          if (need) {
            const Rec4 q = rec[nb];
            const V3<double> n64 = {(double)q.x - p64x, (double)q.y - p64y, (double)q.z - p64z};
            const double d64 = dot(n64, n64);
            if (fabs(d64 - 4.0 * r64) <= 1e-12 * d64) {
              st = VOTESS_CELL_UNRESOLVED;
              kneed = -1 - m;
              run = false;
            } else if (d64 * kDmargin > 4.0 * r64) {
              st = VOTESS_CELL_CERTIFIED;
              kneed = m + 1;
              run = false;
            }
            ++nrecheck;
          }
        }
      }
      const R nx = shfl_t(cx_, gb + i), ny = shfl_t(cy_, gb + i), nz = shfl_t(cz_, gb + i);
      const R d2 = dist2_nc(nx, ny, nz);
      const bool ap = run && ((pendb >> i) & 1u);
      const bool did = apply_plane(ap, nx, ny, nz, R(0.5) * d2, d2, nb, m);
      // on past plane m; if it cut, its own distance may already certify the
      // cell that it left (with a list of m + 1)
      again = ap && did;
      if (run) cur = again ? i : i + 1;
      pendb &= ~(run ? 1u << i : 0u);
    }
  }
  // ---- end of the list: certified if the list holds all others
  if (st == ST_RUN) {
    if (a.k >= a.n - 1) {
      st = VOTESS_CELL_CERTIFIED;
      kneed = a.k;
    } else {
      st = VOTESS_CELL_RADIUS;
    }
  }
  if constexpr (!STREAM && TMAX == kListVert) {
    if (a.save) {  // the stream kernel goes on from here
      const bool sv = have && st == VOTESS_CELL_RADIUS;
      int* w = a.nbr + (size_t)row * a.max_nbr;
      unsigned short* tr = (unsigned short*)(w + kStateTri);
      if (sv)
        for (int f = j; f < 32; f += L) w[f] = pid(f);
      int cnt = 0;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const unsigned u = tri[vb + j + L * s];
        const bool on = sv && u != kEmpty;
        const unsigned gbits = gballot(on);
        if (on)
          tr[cnt + __popc(gbits & below)] = (unsigned short)u;
        cnt += __popc(gbits);
      }
      if (sv && j == 0) {
        w[kStateAlive] = (int)(unsigned)alive;
        w[kStateCount] = cnt;
      }
    }
  }

  // ---- stream phase: a cell its list did not certify keeps clipping by grid
  // rings around its seed, restricted to the bounding box of its "flower" (the
  // union of the balls centred at its vertices that pass through the seed: a
  // point outside every such ball is on the inner side of its bisector at
  // every vertex, so it cannot cut; flowers only shrink as the cell does).
  // Points already in the list are skipped by their (d^2, sorted index) key,
  // points beyond the security radius by d^2 > 4 R^2.  The cell is final once
  // the scanned block of rings contains the flower box.
  // With no list at all (k = 0) every cell starts here, at ring 0: the
  // fused form, with no k-NN pass and no list in memory.
  if constexpr (STREAM) {
    const bool nolist = a.k == 0;
    const int ik0 = (have && st == VOTESS_CELL_RADIUS && !nolist) ? klist[a.k - 1] : -1;
    const bool strm = have && st == VOTESS_CELL_RADIUS && (nolist || ik0 >= 0);  // a full list that did not certify
    if (strm) st = ST_RUN;
    streamed = strm;
    const GridDev& Gd = a.grid;
    const int cx = axis_cell(p64x, Gd.lo0, Gd.ih0, Gd.g0);
    const int cy = axis_cell(p64y, Gd.lo1, Gd.ih1, Gd.g1);
    const int cz = axis_cell(p64z, Gd.lo2, Gd.ih2, Gd.g2);
    const double gmarg = 1e-9 * fmax(Gd.hi0 - Gd.lo0, fmax(Gd.hi1 - Gd.lo1, Gd.hi2 - Gd.lo2));
    R dk2 = R(-1);  // no list: every candidate lies beyond it
    int ik = -1;
    if (strm && !nolist) {
      ik = ik0;
      const Rec4 q = rec[ik];
      dk2 = dist2_nc((R)q.x - px, (R)q.y - py, (R)q.z - pz);
    }
    // A vertex whose widened ball reaches less than the list's ball from the
    // seed (twice its radius below that ball's) can only hold list members:
    // the flower box and the reach list leave it out.
    const double dk2in = (double)dk2 * (1.0 - 1e-6);
    const R rlim = dk2in > 0.0 ? (R)(0.5 * sqrt(dk2in) * (1.0 - 1e-6)) : R(-1);
    // Boxes of candidates, and candidates, are tested in the clip's precision,
    // relative to the seed; the bounds of boxes are widened by gmarg and, in
    // float, rounded outward.  (Float tests would lose the double clip points
    // that cut by less than a float can tell: a cell a thousand times as long as
    // wide and smaller than 1e-8 of the box lost a fifth of those that cut its
    // tip by 1e-10 of the cell.)
    struct Box {
      R x0, x1, y0, y1, z0, z1;
    };
    auto round_out = [&](double x0, double x1, double y0, double y1, double z0, double z1) -> Box {
      if constexpr (RECHECK) {
        auto next = [](float f, int up) -> float {  // the next float below (up = -1) or above (+1) f
          const int b = __float_as_int(f);
          return f == 0.0f ? up * FLT_MIN : __int_as_float(b + (b < 0 ? -up : up));
        };
        auto lo = [&](double v) -> float { const float f = (float)v; return (double)f > v ? next(f, -1) : f; };
        auto hi = [&](double v) -> float { const float f = (float)v; return (double)f < v ? next(f, 1) : f; };
        return {lo(x0), hi(x1), lo(y0), hi(y1), lo(z0), hi(z1)};
      } else {
        return {x0, x1, y0, y1, z0, z1};
      }
    };
    // A box that lies inside the list's ball holds list members only: every
    // point in it is closer than the list's last one even after the rounding
    // of d^2.
    auto in_list_ball = [&](double x0, double x1, double y0, double y1, double z0, double z1) -> bool {
      return fmax(x0 * x0, x1 * x1) + fmax(y0 * y0, y1 * y1) + fmax(z0 * z0, z1 * z1) < dk2in;
    };
    // The reach list: the vertices whose ball leaves the list's ball, as
    // (position, ball radius).  A point cuts the cell iff it lies in the ball
    // of some vertex v through the seed (centre v, radius |v|), so a box that
    // meets none of these balls holds no cutting point, and a candidate is
    // tested against these vertices alone.  Rebuilt after a cut; should it not
    // fit, every test passes (reach_all), which costs time only.
    const int rvb = STREAM ? g * kReach : 0;
    auto ball = [&](int i) -> Ball {
      if constexpr (kCopies) {
        return reachv[rvb + i];
      } else {
        const int t = vb + reachs[rvb + i];
        return {vx[t], vy[t], vz[t], reachr[rvb + i]};
      }
    };
    int nrv = 0;
    R rmax = R(0);  // double clip: the largest |v|
    bool reach_ok = false, reach_all = false;
    auto reach = [&]() {
      int n = 0;
      if constexpr (!RECHECK) rmax = sqrt(R2);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (L * s >= H) continue;
        const int t = j + L * s;
        float e;
        const V3<R> v = vget_err(t, e);
        const R r = ball_rad(v.x, v.y, v.z, e);
        const bool on = tri[vb + t] != kEmpty && r >= rlim;
        const unsigned gbits = gballot(on);
        const int w = n + __popc(gbits & below);
        if (on && w < kReach) {
          if constexpr (kCopies) {
            reachv[rvb + w] = {v.x, v.y, v.z, r};
          } else {
            reachr[rvb + w] = r;
            reachs[rvb + w] = (unsigned char)t;
          }
        }
        n += __popc(gbits);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      reach_all = n > kReach;
      nrv = min(n, kReach);
      reach_ok = true;
    };
    auto meets = [](const Box& b, const Ball& v) -> bool {
      const R gx = fmax(R(0), fmax(b.x0 - v.x, v.x - b.x1)), gy = fmax(R(0), fmax(b.y0 - v.y, v.y - b.y1)),
              gz = fmax(R(0), fmax(b.z0 - v.z, v.z - b.z1));
      return gx * gx + gy * gy + gz * gz <= v.r * v.r;
    };
    // The flower box (of the union of those balls), in coordinates and in grid
    // cells.  Candidates are enumerated inside it, ring by ring of grid cells.
    Enum& E_ = senum[STREAM ? g : 0];
    int &fb0 = E_.fb0, &fb1 = E_.fb1, &fb2 = E_.fb2, &fb3 = E_.fb3, &fb4 = E_.fb4, &fb5 = E_.fb5;
    double* fwb = fwbox + (STREAM ? g * 6 : 0);
    bool flower_ok = false;
    auto flower_box = [&]() {
      double mn0 = 1e300, mn1 = 1e300, mn2 = 1e300, mx0 = -1e300, mx1 = -1e300, mx2 = -1e300;
      for (int t = j; t < H; t += L) {
        if (tri[vb + t] == kEmpty) continue;
        float e;
        const V3<R> v = vget_err(t, e);
        const R rad = ball_rad(v.x, v.y, v.z, e);
        if (rad < rlim) continue;
        const double X = v.x, Y = v.y, Z = v.z, r = rad;
        mn0 = fmin(mn0, X - r); mx0 = fmax(mx0, X + r);
        mn1 = fmin(mn1, Y - r); mx1 = fmax(mx1, Y + r);
        mn2 = fmin(mn2, Z - r); mx2 = fmax(mx2, Z + r);
      }
#pragma unroll
      for (int o = 1; o < L; o <<= 1) {
        mn0 = fmin(mn0, red_step(mn0, o)); mx0 = fmax(mx0, red_step(mx0, o));
        mn1 = fmin(mn1, red_step(mn1, o)); mx1 = fmax(mx1, red_step(mx1, o));
        mn2 = fmin(mn2, red_step(mn2, o)); mx2 = fmax(mx2, red_step(mx2, o));
      }
      if (mn0 > mx0) {  // every ball inside the list's: the seed's own cell closes the scan
        mn0 = mx0 = mn1 = mx1 = mn2 = mx2 = 0.0;
      }
      const double fw0 = p64x + mn0 - gmarg, fw1 = p64x + mx0 + gmarg;
      const double fw2 = p64y + mn1 - gmarg, fw3 = p64y + mx1 + gmarg;
      const double fw4 = p64z + mn2 - gmarg, fw5 = p64z + mx2 + gmarg;
      if (j == 0) {
        fwb[0] = fw0; fwb[1] = fw1; fwb[2] = fw2; fwb[3] = fw3; fwb[4] = fw4; fwb[5] = fw5;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      fb0 = axis_cell(fw0, Gd.lo0, Gd.ih0, Gd.g0);
      fb1 = axis_cell(fw1, Gd.lo0, Gd.ih0, Gd.g0);
      fb2 = axis_cell(fw2, Gd.lo1, Gd.ih1, Gd.g1);
      fb3 = axis_cell(fw3, Gd.lo1, Gd.ih1, Gd.g1);
      fb4 = axis_cell(fw4, Gd.lo2, Gd.ih2, Gd.g2);
      fb5 = axis_cell(fw5, Gd.lo2, Gd.ih2, Gd.g2);
      flower_ok = true;
    };
    // (Row parts taken one by one by the whole group, with a vertex list each,
    // cost most of a streamed cell: of 2^20 uniform points 82k stream and see
    // 52 parts, 16 vertex lists, 10 batches and 45 candidates each; the stream
    // kernel took 3.16 ms for them, with the parts spread over the lanes and
    // the small ones merged into batches 1.32 ms; 16M clustered points, 4.9M
    // streamed cells: 190 and 129 ms.)
    // The ring's row parts (z, y, then the row's x-run on the ring's faces, or
    // its two end cells), by ordinal: tested and looked up one per lane; the
    // ones that can hold a cutting point are listed in order.  A part of at
    // most kSubMin points holds no dense cell and is listed as its points
    // [x, x + y); another one as -1 - ordinal in y, to be walked by itself.
    int &rr = E_.rr, &pq = E_.pq, &np = E_.np, &zlo = E_.zlo, &ylo = E_.ylo, &nyr = E_.nyr, &rln = E_.rln, &rlp = E_.rlp;
    rr = -1; pq = 0; np = 0; zlo = 0; ylo = 0; nyr = 1; rln = 0; rlp = 0;
    int2* rowl = rowlist + (STREAM ? g * L : 0);
    auto row_part = [&](int q, int& x0, int& x1, int& y, int& z) -> bool {
      const int row = q >> 1;
      const int zi = row / nyr;
      z = zlo + zi;
      y = ylo + (row - zi * nyr);
      const int dz = z - cz, dy = y - cy;
      if (dz == rr || dz == -rr || dy == rr || dy == -rr) {  // on a face of the ring
        x0 = max(cx - rr, fb0);
        x1 = min(cx + rr, fb1);
        return !(q & 1) && x0 <= x1;
      }
      x0 = x1 = (q & 1) ? cx + rr : cx - rr;
      return (q & 1) ? x1 <= fb1 : x0 >= fb0;
    };
    // can row part [x0, x1] of row (y, z) hold a cutting point: not inside the
    // list's ball, and meeting the ball of a vertex in reach?  (one part per
    // lane, or the same one in every lane)
    auto part_reached = [&](int x0, int x1, int y, int z) -> bool {
      const double ax = Gd.lo0 + x0 * Gd.h0 - p64x, ay = Gd.lo1 + y * Gd.h1 - p64y, az = Gd.lo2 + z * Gd.h2 - p64z;
      const double bx = ax + (x1 - x0 + 1) * Gd.h0, by = ay + Gd.h1, bz = az + Gd.h2;
      const double m = 2.0 * gmarg;  // (also covers the rounding of these sums)
      if (in_list_ball(ax - m, bx + m, ay - m, by + m, az - m, bz + m)) return false;
      const Box b = round_out(ax - m, bx + m, ay - m, by + m, az - m, bz + m);
      bool any = reach_all;
#pragma unroll(kAhead)
      for (int i = 0; i < nrv; ++i) any = any || meets(b, ball(i));
      return any;
    };
    int jcur = 0, jend = 0;
    // the x-run being split at dense cells, and the sub-block of the dense
    // cell being scanned (sub-cells that meet the flower box)
    int &rx = E_.rx, &rx1 = E_.rx1, &rrow = E_.rrow, &yy = E_.yy, &zz = E_.zz;
    rx = 1; rx1 = 0; rrow = 0; yy = 0; zz = 0;
    // dense cell rows: z and y outward from the seed's row (0, +1, -1, +2, ...)
    int &dm = E_.dm, &dm0 = E_.dm0, &dm1 = E_.dm1, &dm2 = E_.dm2, &dbase = E_.dbase, &dsx0 = E_.dsx0, &dsx1 = E_.dsx1,
        &dsy0 = E_.dsy0, &dsy1 = E_.dsy1, &dsz0 = E_.dsz0, &dsz1 = E_.dsz1;
    dm = 0; dm0 = 0; dm1 = 0; dm2 = 0; dbase = 0; dsx0 = 0; dsx1 = -1; dsy0 = 0; dsy1 = -1; dsz0 = 0; dsz1 = -1;
    int &dq1 = E_.dq1, &dq2 = E_.dq2, &kyn = E_.kyn, &kzn = E_.kzn;
    dq1 = 0; dq2 = 0; kyn = 0; kzn = 0;
    // next sub-row ordinal, their count; listed ranges, next one
    int &dq = E_.dq, &dqn = E_.dqn, &srn = E_.srn, &srp = E_.srp;
    dq = 0; dqn = 0; srn = 0; srp = 0;
    int& dsto = E_.dsto;  // the dense cell's sub-grid record: a.sub.start + dsto
    dsto = 0;
    // entries of the reach list whose ball meets the dense cell's sub-block
    // (valid for the vertices they were listed for)
    unsigned char* rd = relD + (STREAM ? g * kReach : 0);
    int nD = 0;
    bool okD = false;
    // can sub-row (sy, sz) of the dense cell's sub-block hold a cutting point:
    // not inside the list's ball, and (while the dense cell's vertex list is
    // valid) meeting the ball of a listed vertex?  (one sub-row per lane)
    auto sub_row_relevant = [&](int sy, int sz) -> bool {
      const double* dgp = dgeo + g * 3;
      const SubCell sc = sub_cell(a.sub.start + dsto);
      const double cxl = Gd.lo0 + (rx - 1) * Gd.h0, cyl = Gd.lo1 + yy * Gd.h1, czl = Gd.lo2 + zz * Gd.h2;
      const double X0 = dsx0 == 0 ? cxl : sc.lo0 + dsx0 * dgp[0];
      const double X1 = dsx1 == dm0 - 1 ? cxl + Gd.h0 : sc.lo0 + (dsx1 + 1) * dgp[0];
      const double Y0 = sy == 0 ? cyl : sc.lo1 + sy * dgp[1];
      const double Y1 = sy == dm1 - 1 ? cyl + Gd.h1 : sc.lo1 + (sy + 1) * dgp[1];
      const double Z0 = sz == 0 ? czl : sc.lo2 + sz * dgp[2];
      const double Z1 = sz == dm2 - 1 ? czl + Gd.h2 : sc.lo2 + (sz + 1) * dgp[2];
      const double ax = X0 - p64x - gmarg, bx = X1 - p64x + gmarg, ay = Y0 - p64y - gmarg, by = Y1 - p64y + gmarg,
                   az = Z0 - p64z - gmarg, bz = Z1 - p64z + gmarg;
      if (in_list_ball(ax, bx, ay, by, az, bz)) return false;
      const Box b = round_out(ax, bx, ay, by, az, bz);
      bool any = !okD || reach_all;
#pragma unroll(kAhead)
      for (int i = 0; i < nD; ++i) any = any || meets(b, ball(rd[i]));
      return any;
    };
    bool rdense = false;  // the current range lies in a dense cell
    // The next batch of up to L candidates, one per lane: jj, and tag, the
    // order among the ranges of the batch (planes of a lower tag are applied
    // first).  False when the scan is complete.  (Each step is taken by a whole
    // group.)
    auto next_batch = [&](int& jj, int& tag) -> bool {
      jj = -1;
      tag = 0;
      for (;;) {
        if (jcur < jend) {
          // the rest of the current range, then (in a dense cell) the
          // following listed sub-rows
          int nb = 0;
          for (;;) {
            const int take = min(L - nb, jend - jcur);
            if (j >= nb && j < nb + take) jj = jcur + (j - nb);
            nb += take;
            jcur += take;
            if (nb == L || !rdense || srp >= srn) return true;
            const int2 rg = srl[g * L + srp];
            ++srp;
            jcur = dbase + rg.x;
            jend = dbase + rg.y;
          }
        }
        if (dm > 0) {
          // the dense cell's sub-rows inside the flower box, one x-run
          // each, rows nearer the seed first: the next L of them are
          // tested and their ranges read at once, one per lane, and the
          // non-empty ranges listed
          if (srp >= srn) {
            if (dq >= dqn) {
              dm = 0;
              continue;
            }
            const int q = dq + j;
            dq += L;
            bool keep = false;
            int lo = 0, hi = 0;
            if (q < dqn) {
              const int qz = q / kyn, qy = q - qz * kyn;
              const int sz = dq2 + ((qz & 1) ? (qz + 1) >> 1 : -(qz >> 1));
              const int sy = dq1 + ((qy & 1) ? (qy + 1) >> 1 : -(qy >> 1));
              if (sz >= dsz0 && sz <= dsz1 && sy >= dsy0 && sy <= dsy1 && sub_row_relevant(sy, sz)) {
                const int rowb = kSubHead + dm0 * (sy + dm1 * sz);
                lo = a.sub.start[dsto + rowb + dsx0];
                hi = a.sub.start[dsto + rowb + dsx1 + 1];
                keep = lo < hi;
              }
            }
            const unsigned kb = gballot(keep);
            if (keep) srl[g * L + __popc(kb & below)] = make_int2(lo, hi);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            srn = __popc(kb);
            srp = 0;
            continue;
          }
          const int2 rg = srl[g * L + srp];
          ++srp;
          jcur = dbase + rg.x;
          jend = dbase + rg.y;
          rdense = true;
          continue;
        }
        if (rx <= rx1) {
          int xe = rx1 + 1;
          if (a.sub.info) {
            // the stretch of cells without sub-grids: the group reads L
            // consecutive cells' records at once and ends it at the
            // first dense one
            xe = rx;
            for (;;) {
              const int xc = xe + j;
              const bool dn = xc <= rx1 && is_dense(a.sub.info[rrow + xc]);
              const unsigned dmask = gballot(dn);
              if (dmask) {
                xe += __ffs(dmask) - 1;
                break;
              }
              xe += L;
              if (xe > rx1) {
                xe = rx1 + 1;
                break;
              }
            }
          }
          if (xe > rx) {
            jcur = a.cell_start[rrow + rx];
            jend = a.cell_start[rrow + xe];
            rx = xe;
            rdense = false;
            continue;
          }
          // dense cell rx: its sub-cells inside the flower box
          const int2 info = a.sub.info[rrow + rx];
          const SubCell sc = sub_cell(sub_record(a.sub, info));
          dsx0 = sub_axis(fwb[0], sc.lo0, sc.ih0, sc.m0);
          dsx1 = sub_axis(fwb[1], sc.lo0, sc.ih0, sc.m0);
          dsy0 = sub_axis(fwb[2], sc.lo1, sc.ih1, sc.m1);
          dsy1 = sub_axis(fwb[3], sc.lo1, sc.ih1, sc.m1);
          dsz0 = sub_axis(fwb[4], sc.lo2, sc.ih2, sc.m2);
          dsz1 = sub_axis(fwb[5], sc.lo2, sc.ih2, sc.m2);
          {
            // the sub-block's box (edge sub-cells reach the cell's faces)
            const double cxl = Gd.lo0 + rx * Gd.h0, cyl = Gd.lo1 + yy * Gd.h1, czl = Gd.lo2 + zz * Gd.h2;
            const double w0 = 1.0 / sc.ih0, w1 = 1.0 / sc.ih1, w2 = 1.0 / sc.ih2;
            const double X0 = dsx0 == 0 ? cxl : sc.lo0 + dsx0 * w0;
            const double X1 = dsx1 == sc.m0 - 1 ? cxl + Gd.h0 : sc.lo0 + (dsx1 + 1) * w0;
            const double Y0 = dsy0 == 0 ? cyl : sc.lo1 + dsy0 * w1;
            const double Y1 = dsy1 == sc.m1 - 1 ? cyl + Gd.h1 : sc.lo1 + (dsy1 + 1) * w1;
            const double Z0 = dsz0 == 0 ? czl : sc.lo2 + dsz0 * w2;
            const double Z1 = dsz1 == sc.m2 - 1 ? czl + Gd.h2 : sc.lo2 + (dsz1 + 1) * w2;
            const double ax = X0 - p64x - gmarg, bx = X1 - p64x + gmarg, ay = Y0 - p64y - gmarg,
                         by = Y1 - p64y + gmarg, az = Z0 - p64z - gmarg, bz = Z1 - p64z + gmarg;
            nD = 0;
            okD = true;
            bool hit = false;
            if (!in_list_ball(ax, bx, ay, by, az, bz)) {
              const Box b = round_out(ax, bx, ay, by, az, bz);
              for (int i0 = 0; i0 < nrv; i0 += L) {
                const bool on = i0 + j < nrv && meets(b, ball(i0 + j));
                const unsigned gbits = gballot(on);
                if (on) rd[nD + __popc(gbits & below)] = (unsigned char)(i0 + j);
                nD += __popc(gbits);
              }
              hit = nD > 0 || reach_all;
            }
            if (j == 0) {
              double* dgp = dgeo + g * 3;
              dgp[0] = w0; dgp[1] = w1; dgp[2] = w2;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            dm = hit ? 1 : 0;
          }
          if (dm) {
            dsto = info.x;
            dbase = a.cell_start[rrow + rx];
            dm0 = sc.m0;
            dm1 = sc.m1;
            dm2 = sc.m2;
            dq1 = min(max(sub_axis(p64y, sc.lo1, sc.ih1, sc.m1), dsy0), dsy1);
            dq2 = min(max(sub_axis(p64z, sc.lo2, sc.ih2, sc.m2), dsz0), dsz1);
            // offsets 0, +1, -1, ... up to the farther end of each range
            kyn = 2 * max(dq1 - dsy0, dsy1 - dq1) + 1;
            kzn = 2 * max(dq2 - dsz0, dsz1 - dq2) + 1;
            dq = 0;
            dqn = kyn * kzn;
            srn = srp = 0;
          }
          ++rx;
          continue;
        }
        if (rlp < rln) {
          // whole listed parts while they fit the batch
          int nb = 0;
          while (rlp < rln) {
            const int2 e = rowl[rlp];
            if (e.y < 0 || nb + e.y > L) break;
            if (j >= nb && j < nb + e.y) {
              jj = e.x + (j - nb);
              tag = rlp;
            }
            nb += e.y;
            ++rlp;
          }
          rdense = false;
          if (nb > 0) return true;
          // a part with more points: tested again for the vertices as they are
          int x0, x1;
          row_part(-1 - rowl[rlp].y, x0, x1, yy, zz);
          ++rlp;
          if (part_reached(x0, x1, yy, zz)) {
            rrow = Gd.g0 * (yy + Gd.g1 * zz);
            rx = x0;
            rx1 = x1;
          }
          continue;
        }
        if (pq < np) {
          const int q = pq + j;
          pq += L;
          bool keep = false;
          int lo = 0, len = 0, x0, x1, y, z;
          if (q < np && row_part(q, x0, x1, y, z) && part_reached(x0, x1, y, z)) {
            const int row = Gd.g0 * (y + Gd.g1 * z);
            lo = a.cell_start[row + x0];
            len = a.cell_start[row + x1 + 1] - lo;
            keep = len > 0;
          }
          const unsigned kb = gballot(keep);
          if (keep) rowl[__popc(kb & below)] = make_int2(lo, len <= kSubMin ? len : -1 - q);
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          rln = __popc(kb);
          rlp = 0;
          continue;
        }
        // ring rr finished (or none yet): final when the block contains the flower box
        if (!flower_ok) flower_box();
        if (rr >= 0 && cx - rr <= fb0 && cx + rr >= fb1 && cy - rr <= fb2 && cy + rr >= fb3 && cz - rr <= fb4 &&
            cz + rr >= fb5)
          return false;
        ++rr;
        zlo = max(cz - rr, fb4);
        ylo = max(cy - rr, fb2);
        nyr = min(cy + rr, fb3) - ylo + 1;
        pq = 0;
        np = nyr > 0 ? max(0, min(cz + rr, fb5) - zlo + 1) * nyr * 2 : 0;
      }
    };
    unsigned pend = 0;
    int myj = -1, mytag = 0;
    R myx = R(0), myy = R(0), myz = R(0), myd2 = R(0);
    const R skip_scale = RECHECK ? R(1) - R(2e-6) : R(1) - R(1e-12);
    // can this lane's candidate cut: within twice the radius, and some vertex
    // in reach on the far side of the bisector, up to a bound on the plane
    // test's own uncertainty (and on the arithmetic here)?
    auto may_cut = [&]() -> bool {
      if (!(myd2 * skip_scale <= R(4) * (RECHECK ? (R)R2up : R2))) return false;
      if (reach_all) return true;
      const R c = R(0.5) * myd2;
      R far = -c;
      if (rdense && okD) {
#pragma unroll(kAhead)
        for (int i = 0; i < nD; ++i) {
          const Ball v = ball(rd[i]);
          far = fmax(far, myx * v.x + myy * v.y + myz * v.z);
        }
      } else {
#pragma unroll(kAhead)
        for (int i = 0; i < nrv; ++i) {
          const Ball v = ball(i);
          far = fmax(far, myx * v.x + myy * v.y + myz * v.z);
        }
      }
      R w;
      if constexpr (RECHECK) w = (wv + 2e-6f) * (c + __builtin_amdgcn_sqrtf(2.0f * c) * __builtin_amdgcn_sqrtf(R2up));
      else w = R(1e-12) * (c + (fabs(myx) + fabs(myy) + fabs(myz)) * rmax);
      return !(far < c - w);
    };
    while (__any(strm && st == ST_RUN)) {
      const bool act = strm && st == ST_RUN;
      // after a cut, the batch's other candidates are tested again together
      // (rather than applied one by one: a cut leaves few of them)
      if (act && pend != 0u && !reach_ok) {
        reach();
        pend &= gballot(((pend >> j) & 1u) && may_cut());
      }
      // the group's next batch with a candidate that may cut (group-uniform
      // loop), beyond the list
      while (act && pend == 0u) {
        if (!reach_ok) reach();
        if (!next_batch(myj, mytag)) {
          st = VOTESS_CELL_CERTIFIED;
          kneed = a.k + 1;
          break;
        }
        bool pass = false;
        if (myj >= 0 && myj != sid) {
          const Rec4 q = rec[myj];
          myx = (R)q.x - px;
          myy = (R)q.y - py;
          myz = (R)q.z - pz;
          myd2 = dist2_nc(myx, myy, myz);
          pass = (myd2 > dk2 || (myd2 == dk2 && myj > ik)) && may_cut();
        }
        pend = gballot(pass);
      }
      // nearest pending candidate of the group, range by range
      bool run2 = act && st == ST_RUN && pend != 0u;
      int bl = run2 ? __ffs(pend) - 1 : j;
      if (__any(run2 && (pend & (pend - 1u)) != 0u)) {
        const bool on = run2 && ((pend >> j) & 1u);
        R best = on ? myd2 : R(3.0e38);
        int bt = on ? mytag : 0x7FFFFFFF;
        bl = j;
#pragma unroll
        for (int o = 1; o < L; o <<= 1) {
          const R ob = red_step(best, o);
          const int ot = red_step(bt, o), ol = red_step(bl, o);
          if (ot < bt || (ot == bt && (ob < best || (ob == best && ol < bl)))) { best = ob; bt = ot; bl = ol; }
        }
      }
      const int nb2 = __shfl(myj, gb + bl, 64);
      const R nx = shfl_t(myx, gb + bl), ny = shfl_t(myy, gb + bl), nz = shfl_t(myz, gb + bl);
      const R d2 = dist2_nc(nx, ny, nz), c = R(0.5) * d2;
      if (run2) {
        pend &= ~(1u << bl);
        // the radius may have shrunk since the batch was filtered
        if (d2 * skip_scale > R(4) * (RECHECK ? (R)R2up : R2)) run2 = false;
      }
      if (apply_plane(run2, nx, ny, nz, c, d2, nb2, -1)) reach_ok = okD = flower_ok = false;
    }
  }

  // ---- outputs
  const bool cert = have && st == VOTESS_CELL_CERTIFIED;
  // volume: corner terms in double.  `exact` takes vertices and planes in
  // double from the inputs (float path, ill-conditioned cells only).
  // Anchor of edge f^g: the point of the line nearest the seed,
  // (c_f (n_g x d) - c_g (n_f x d)) / |d|^2 with d = n_f x n_g.  Its error
  // grows like 1/sin of the angle between the planes; a solve of the 2x2 Gram
  // system would square that, which shows on the faces of nearly parallel
  // neighbours.
  auto anchor = [&](const V3<double>& nf, double cf, const V3<double>& ng, double cg) -> V3<double> {
    const V3<double> d = cross(nf, ng);
    const V3<double> gd = cross(ng, d), fd = cross(nf, d);
    const double inv = 1.0 / dot(d, d);
    return {(cf * gd.x - cg * fd.x) * inv, (cf * gd.y - cg * fd.y) * inv, (cf * gd.z - cg * fd.z) * inv};
  };
  // the three planes and the position of vertex slot t, in double: cached,
  // or (exact) planes from the exact inputs, or (refined) cached or exact
  // planes with the vertex solved and refined in double
  auto corner_geom = [&](unsigned u, int t, bool exact, V3<double>& na, double& ca, V3<double>& nb_, double& cb,
                         V3<double>& nc, double& cc, V3<double>& v, bool refined = false) {
    const int A = TC::a(u), B = TC::b(u), C = TC::c(u);
    if (exact) {
      plane64(A, na, ca);
      plane64(B, nb_, cb);
      plane64(C, nc, cc);
      v = refined ? solve3_refined(na, ca, pid(A) >= 0, nb_, cb, pid(B) >= 0, nc, cc, pid(C) >= 0)
                  : solve3<RECHECK>(na, ca, nb_, cb, nc, cc);
    } else {
      V3<R> ra, rb, rc;
      R da, db, dc;
      pget(A, ra, da);
      pget(B, rb, db);
      pget(C, rc, dc);
      na = {(double)ra.x, (double)ra.y, (double)ra.z};
      nb_ = {(double)rb.x, (double)rb.y, (double)rb.z};
      nc = {(double)rc.x, (double)rc.y, (double)rc.z};
      ca = (double)da;
      cb = (double)db;
      cc = (double)dc;
      if (refined) {
        // bisector offsets are taken exactly only where the cached plane holds
        // the exact normal (double planes)
        constexpr bool kExactN = sizeof(R) == 8;
        v = solve3_refined(na, ca, kExactN && pid(A) >= 0, nb_, cb, kExactN && pid(B) >= 0, nc, cc,
                           kExactN && pid(C) >= 0);
      } else {
        const V3<R> w = vget(t);
        v = {(double)w.x, (double)w.y, (double)w.z};
      }
    }
  };
  // One pass over the corners, a vertex per lane: the volume's terms and, with
  // `faces`, the centroid's moments and the face areas.
  // Cell centroid: the corner terms of the volume split into signed
  // tetrahedra from the seed, (0, F_f, v, e_fh) and (0, F_f, e_fg, v); the
  // first moment of each is its volume times the mean of its corners.
  // Face areas: a face is the fan of the volume's corner terms: the corner of
  // vertex v on face f, between edges f^g and f^h, spans the area
  // n_f . (v x (e_fh - e_fg)) / (2 |n_f|).  Lane j sums the faces of plane
  // slots j, j+L, ..., the slots it writes to the neighbour list below: the
  // lanes' corners go round the group, so each face sums its corners in slot
  // order and every corner is computed once.  Clip with faces, in double, 20k
  // uniform points: 0.35 ms, of which faces 0.03; float, 1.2M filament points:
  // 45.6 ms.  (0.63 and 58.0 with a pass of its own for each output, and each
  // lane computing the corners of its faces among all vertices.)
  constexpr int FO = PMAX / L;
  static_assert(FO * L == PMAX, "plane slots split evenly over the lanes");
  double farea[FO], w6 = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
#pragma unroll
  for (int q = 0; q < FO; ++q) farea[q] = 0.0;
  auto corners = [&](bool on, bool exact, bool faces) -> double {
    double acc = 0.0;
    if (on) {
      for (int t0 = 0; t0 < H; t0 += L) {
        const int t = t0 + j;
        const unsigned u = t < H ? (unsigned)tri[vb + t] : kEmpty;
        double xa = 0.0, xb = 0.0, xc = 0.0;
        if (u != kEmpty) {
          V3<double> na, nb_, nc, v;
          double ca, cb, cc;
          // double planes: every vertex refined once (a vertex of nearly
          // parallel planes is otherwise off by its conditioning times u R)
          corner_geom(u, t, exact, na, ca, nb_, cb, nc, cc, v, exact || sizeof(R) == 8);
          const V3<double> eab = anchor(na, ca, nb_, cb), ebc = anchor(nb_, cb, nc, cc), eca = anchor(nc, cc, na, ca);
          const double qa = dot(na, na), qb = dot(nb_, nb_), qc = dot(nc, nc);
          const double fa = ca / qa, fb = cb / qb, fc = cc / qc;
          const V3<double> Fa = {fa * na.x, fa * na.y, fa * na.z};
          const V3<double> Fb = {fb * nb_.x, fb * nb_.y, fb * nb_.z};
          const V3<double> Fc = {fc * nc.x, fc * nc.y, fc * nc.z};
          const V3<double> wa = cross(v, V3<double>{eca.x - eab.x, eca.y - eab.y, eca.z - eab.z});
          const V3<double> wb = cross(v, V3<double>{eab.x - ebc.x, eab.y - ebc.y, eab.z - ebc.z});
          const V3<double> wc = cross(v, V3<double>{ebc.x - eca.x, ebc.y - eca.y, ebc.z - eca.z});
          acc += dot(Fa, wa);
          acc += dot(Fb, wb);
          acc += dot(Fc, wc);
          if (faces) {
            if (a.centroid) {
              auto tet = [&](const V3<double>& x, const V3<double>& y, const V3<double>& z) {
                const double w = dot(x, cross(y, z));
                w6 += w;
                mx += w * (x.x + y.x + z.x);
                my += w * (x.y + y.y + z.y);
                mz += w * (x.z + y.z + z.z);
              };
              tet(Fa, v, eca);
              tet(Fa, eab, v);
              tet(Fb, v, eab);
              tet(Fb, ebc, v);
              tet(Fc, v, ebc);
              tet(Fc, eca, v);
            }
            xa = dot(na, wa) / (2.0 * sqrt(qa));
            xb = dot(nb_, wb) / (2.0 * sqrt(qb));
            xc = dot(nc, wc) / (2.0 * sqrt(qc));
          }
        }
        if (faces && a.area) {
          for (int i = 0; i < L; ++i) {
            const unsigned w = (unsigned)__shfl((int)u, gb + i, 64);
            const double ya = shfl_t(xa, gb + i), yb = shfl_t(xb, gb + i), yc = shfl_t(xc, gb + i);
            const int A = TC::a(w), B = TC::b(w), C = TC::c(w);
#pragma unroll
            for (int q = 0; q < FO; ++q) {
              const int f = j + q * L;
              farea[q] += (A == f ? ya : 0.0) + (B == f ? yb : 0.0) + (C == f ? yc : 0.0);
            }
          }
        }
      }
    }
    return gsumd(acc) / 6.0;
  };
  // Faces are computed in double from vertices solved in double and refined
  // once: with the volume's corners on the FP64 path, with planes from the
  // exact inputs on the float path.
  const bool faces = a.area || a.centroid;
  double vol = corners(cert, false, !RECHECK && faces);
  // Float vertices carry an absolute error ~u R; a cell much thinner than its
  // radius (R^3 > 16 V, i.e. u R^3 / V > 1e-6) cannot get its volume to 1e-5
  // from them, so its outputs are recomputed from vertices solved in double.
  bool refine = false;
  if (RECHECK) {
    refine = cert && (double)R2 * sqrt((double)R2) > 16.0 * vol;
    const bool again = faces ? cert : refine;
    if (__any(again)) {
      const double v2 = corners(again, true, faces);
      if (refine) vol = v2;
    }
  }
  double cmx = 0.0, cmy = 0.0, cmz = 0.0;
  if (a.centroid) {
    const double V6 = gsumd(w6);
    mx = gsumd(mx);
    my = gsumd(my);
    mz = gsumd(mz);
    // moment / volume = (sum w m / 24) / (sum w / 6)
    if (V6 > 0.0) {
      cmx = p64x + mx / (4.0 * V6);
      cmy = p64y + my / (4.0 * V6);
      cmz = p64z + mz / (4.0 * V6);
    }
  }
  // neighbours: alive bisector planes
  int nnb = 0;
  for (int f = j; f < PMAX; f += L) nnb += cert && ((alive >> f) & 1) && pid(f) >= 0;
  int ntot;
  int noff = gexcl(nnb, ntot);
  // vertices
  int vtot = 0, voff = 0;
  if (a.max_vert > 0) {
    int nv = 0;
    for (int t = j; t < H; t += L) nv += cert && tri[vb + t] != kEmpty;
    voff = gexcl(nv, vtot);
  }
  // the cell's status: certified, unless its row is too short for it.  Rows of
  // cells that are not certified stay as they are.
  int fin = st;
  if (cert && (ntot > a.max_nbr || (a.max_vert > 0 && vtot > a.max_vert))) fin = VOTESS_CELL_CAPACITY;
  const bool put = cert && fin == VOTESS_CELL_CERTIFIED;
  if (put) {
#pragma unroll
    for (int q = 0; q < FO; ++q) {
      const int f = j + q * L;
      if (((alive >> f) & 1) && pid(f) >= 0) {
        a.nbr[(size_t)row * a.max_nbr + noff] = pid(f);
        if (a.area) a.area[(size_t)row * a.max_nbr + noff] = farea[q];
        ++noff;
      }
    }
  }
  if (put && a.max_vert > 0) {
    for (int t = j; t < H; t += L) {
      const unsigned u = tri[vb + t];
      if (u == kEmpty) continue;
      const size_t o = ((size_t)row * a.max_vert + voff) * 3;
      const V3<R> w = vget(t);
      V3<double> v = {(double)w.x, (double)w.y, (double)w.z};
      if (refine) v = vertex64(u);
      a.verts[o + 0] = p64x + v.x;
      a.verts[o + 1] = p64y + v.y;
      a.verts[o + 2] = p64z + v.z;
      a.vplanes[o + 0] = pid(TC::a(u));
      a.vplanes[o + 1] = pid(TC::b(u));
      a.vplanes[o + 2] = pid(TC::c(u));
      ++voff;
    }
  }
  if (have && j == 0) {
    a.status[row] = (uint8_t)(fin | (a.rest || ((a.mark >> fin) & 1) ? kLeft : 0));
    a.nbr_count[row] = fin == VOTESS_CELL_CERTIFIED ? ntot : 0;
    a.volume[row] = fin == VOTESS_CELL_CERTIFIED ? vol : 0.0;
    if (a.centroid) {
      const bool ok = fin == VOTESS_CELL_CERTIFIED;
      a.centroid[(size_t)row * 3 + 0] = ok ? cmx : 0.0;
      a.centroid[(size_t)row * 3 + 1] = ok ? cmy : 0.0;
      a.centroid[(size_t)row * 3 + 2] = ok ? cmz : 0.0;
    }
    if (a.kneeded) a.kneeded[row] = max(kneed, 0);
    if (a.r2out) a.r2out[row] = fin == VOTESS_CELL_CERTIFIED ? (RECHECK ? (double)R2up : (double)R2) : 0.0;
    if (a.vcount) a.vcount[row] = fin == VOTESS_CELL_CERTIFIED ? vtot : 0;
  }
  // counters: one addition per wave (all of them meet at one address)
  if (a.counters) {
    const bool lead = have && j == 0;
    auto add = [&](int c, bool v, bool less = false) {
      const unsigned long long b = __ballot(lead && v);
      const unsigned long long by = (unsigned long long)__popcll(b);
      if (lane == 0 && b) atomicAdd(&a.counters[c], less ? 0ull - by : by);
    };
    add(1, fin == VOTESS_CELL_UNRESOLVED);
    const bool word = !((a.mark >> fin) & 1);  // of this launch, on the cell's status
    add(kCapacityCounter, word && fin == VOTESS_CELL_CAPACITY);
    add(kRadiusCounter, word && fin == VOTESS_CELL_RADIUS);
    add(5, streamed);
    add(4, streamed && st == VOTESS_CELL_CERTIFIED);
    if constexpr (RECHECK) {
      add(3, refine && fin == VOTESS_CELL_CERTIFIED);
      int rc = nrecheck;
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) rc += red_step(rc, o);
      rc += __shfl_xor(rc, 16, 64);
      rc += __shfl_xor(rc, 32, 64);
      if (lane == 0 && rc) atomicAdd(&a.counters[0], (unsigned long long)rc);
    }
    // cells that a pass with lists of level[i] would have left, counted by the
    // launch that has the last word on the cell's list: the large kernel for
    // cells that the fast ones cannot hold, except in the first pass, which has no
    // large kernel (so that a cell that the stream phase, after the list, leaves to
    // the large kernel is taken off again).  A cell that is unresolved at a plane
    // of the list's first level[i] would not have been left, but unresolved.
    const bool over = fin == VOTESS_CELL_CAPACITY && PMAX <= 32;
    const bool mine = !resume && !(over && ((a.mark >> fin) & 1));
#pragma unroll
    for (int i = 0; i < kLevels; ++i)
      if (a.level[i]) {
        add(kLevelCounter + i, mine && (fin == VOTESS_CELL_CERTIFIED    ? kneed > a.level[i]
                                        : fin == VOTESS_CELL_UNRESOLVED ? kneed >= 0 || -1 - kneed >= a.level[i]
                                                                        : !over || i == 0));
        if (STREAM && i > 0) add(kLevelCounter + i, resume && over, true);
      }
  }
}

// One wave (= one block) clips `per` cells, one per group.  With `rest`, the
// list kernel has been over the launch's cells and left some: cells that
// outgrew it (taken again from the box) and, when this is the stream kernel,
// cells that their lists did not certify (resumed).
// Marked cells are packed within each 64: the waves that share 64 cells take
// the first ones, the next ones, ..., and most waves find nothing and end.
// (A wave that loops over its cells keeps so many invariants of the loop in
// registers that it spills.)  The marks stay until k_unmark, so that all of
// these waves see the same ones.
// The order of the blocks is ClipGrid's.
// The kernels are held to 3 waves per SIMD, as many as their LDS lets a CU
// hold: with triangles in 16 bits and planes without their offsets a list
// wave takes 13.1 KB (double clip of float points 16.2, of double ones 19.3)
// and a CU holds 12 (10, 8); with 32-bit triangles and offsets 14.9 (22.1) KB
// and 10 (7).  Clip times with those and with these, one stretch of blocks per
// XCD: 3M clustered points in double 58.9 and 51.1 ms, 16M in float 215.9 and
// 202.6 ms, 1M uniform 6.99 and 6.39.
template <typename P, typename R, int L, int TMAX, int PMAX, bool RECHECK, bool STREAM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_clip(ClipArgs a) {
  constexpr int G = 64 / L;
  const ClipGrid grid(a.nc, a.per, a.rest);
  int unit, wave;
  grid.find(blockIdx.x, unit, wave);
  if (unit >= grid.units) return;  // the whole (one-wave) block
  const int lane = threadIdx.x, g = lane / L;
  long long t_idx = (long long)unit * a.per + g;
  bool have = g < a.per && t_idx < a.nc, resume = false;
  if (a.rest) {
    const long long base = (long long)unit * 64;
    int stat = 0;
    if (base + lane < a.nc) stat = a.status[a.out_by_id && a.cells ? (long long)a.cells[base + lane] : base + lane];
    unsigned long long todo = __ballot((stat & kLeft) != 0);
    const int skip = wave * a.per;  // cells that the waves before this one take
    if (__popcll(todo) <= skip) return;
    for (int i = 0; i < skip; ++i) todo &= todo - 1ull;
    int at = -1;
#pragma unroll
    for (int i = 0; i < G; ++i) {  // the i-th of the cells left goes to group i
      if (todo && g == i && i < a.per) at = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
    }
    have = at >= 0;
    t_idx = base + at;
    const int from = __shfl(stat, have ? at : 0, 64);  // by every lane: a shuffle reads active lanes only
    resume = STREAM && have && from == (kLeft | VOTESS_CELL_RADIUS);
  }
  clip_group<P, R, L, TMAX, PMAX, RECHECK, STREAM>(a, have ? t_idx : 0, have, resume);
}

constexpr int kFillWaves = 2048, kRestWaves = 8192;

// takes the marks off again
__global__ void k_unmark(uint8_t* status, const int* cells, int nc) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nc) return;
  uint8_t* p = status + (cells ? (long long)cells[t] : t);
  const uint8_t v = *p;
  if (v & kLeft) *p = v & (uint8_t)~kLeft;
}

template <typename P, typename R, int L, int TMAX, int PMAX, bool RECHECK, bool STREAM>
void launch(ClipArgs ca, bool rest, hipStream_t st) {
  ca.rest = rest;
  // A wave's groups wait on each other wherever they diverge, so that a wave
  // of one cell is done sooner than a wave of several.  Waves are filled only
  // as far as the cells suffice for kFillWaves of them (two per SIMD).  Clip
  // time with full waves, from 2048 and from 4096: 10k clustered points, float
  // 2.87, 2.53 and 2.59 ms; 100k 6.69, 6.08 and 6.21 ms; 8k filament points,
  // double 1.24, 1.14 and 1.28 ms; 8k uniform ones, float 0.26, 0.32 and 0.34.
  // A launch over the cells that are left finds a tenth to two thirds of them,
  // so that its waves are filled from four times as many on (10k clustered
  // points from 2048, 8192 and 16384: 2.57, 2.46 and 2.46 ms; 30k filament
  // points with faces 0.465, 0.466 and 0.496).
  ca.per = 64 / L;
  while (ca.per > 1 && ca.nc / ca.per < (rest ? kRestWaves : kFillWaves)) ca.per /= 2;
  k_clip<P, R, L, TMAX, PMAX, RECHECK, STREAM><<<ClipGrid(ca.nc, ca.per, rest).blocks(), 64, 0, st>>>(ca);
}

template <typename P, typename R, int L, int TMAX, int PMAX, bool RECHECK>
void launch_all(const ClipArgs& ca, bool rest, hipStream_t st) {
  if (ca.stream)
    launch<P, R, L, TMAX, PMAX, RECHECK, true>(ca, rest, st);
  else
    launch<P, R, L, TMAX, PMAX, RECHECK, false>(ca, rest, st);
}

// The fast kernels.  Lists are clipped by 8 lanes per cell: list cells are
// bound by vector instructions, and 8 lanes waste fewer of them than 16 (a cut
// makes about 6 new vertices); 48 vertex slots let more waves fit a CU.  A
// stream cell waits on loads, and its batches of candidates fill 16 lanes; 48
// slots and fewer vertices in reach would let 4 waves fit a SIMD rather than
// 3, but clustered cells overflow them (16M points: 208 -> 312 ms).  Cells that
// outgrow the list kernel share the second launch: in one of their own they
// leave the chip half empty (1.2M filament points: 36.3 ms together, 29.9 and
// 10.2 ms apart).
// Without the stream phase the list kernel does alone where it can: with lists
// of at most kShortList planes, which with the box make no more vertices than it
// has slots for (500k clustered cells by 16 planes: 1.19 ms with a second
// launch that finds nothing and the marks' removal, 1.14 without; 2000 cells 57
// and 54 us), and, with the stream kernel's 64 slots, over few cells, where the
// second launch would wait for a handful that outgrew the first (64 planes: 2000
// cells 201 and 113 us, 32,000 uniform ones 316 and 235, 128,000 728 and 739;
// 32 planes: 8000 cells 252 and 178 us, 32,000 clustered ones 228 and 235).  A
// cell's sums have the same order either way.
constexpr int kShortList = (kListVert + 4) / 2 - 6;  // (f faces make 2 f - 4 vertices)
template <typename P, typename R, bool RECHECK>
votess_status run_fast(ClipArgs ca, bool split, hipStream_t st) {
  if (split && !ca.stream) {
    const bool few = ca.nc < (ca.k > 32 ? 65536 : 32768);
    if (ca.k <= kShortList || few) {
      if (ca.k <= kShortList)
        launch<P, R, kListLanes, kListVert, 32, RECHECK, false>(ca, false, st);
      else
        launch<P, R, kListLanes, 64, 32, RECHECK, false>(ca, false, st);
      VT_HIP(hipGetLastError());
      return VOTESS_OK;
    }
  }
  if (split) {
    ca.save = ca.stream;
    ca.mark = 1 << VOTESS_CELL_CAPACITY | (ca.stream ? 1 << VOTESS_CELL_RADIUS : 0);
    launch<P, R, kListLanes, kListVert, 32, RECHECK, false>(ca, false, st);
    ca.save = ca.mark = 0;
  }
  launch_all<P, R, 16, 64, 32, RECHECK>(ca, split, st);
  if (split)
    k_unmark<<<(unsigned)(((long long)ca.nc + 255) / 256), 256, 0, st>>>(ca.status, ca.out_by_id ? ca.cells : nullptr,
                                                                        ca.nc);
  VT_HIP(hipGetLastError());
  return VOTESS_OK;
}

// The large-capacity kernel.  64 planes make 2 * 64 - 4 = 124 vertices at most
// (a simple polyhedron), so 128 slots hold every cell that the planes let it
// hold; with 256 a wave takes 24 KB and a SIMD holds 1.5 of them.  Clip of 1.2M
// filament points with faces, 33,000 of them here: 45.6 ms with 256 slots, 43.3
// with 128; with 16 lanes per cell 46.6.
template <typename P, typename R, bool RECHECK>
votess_status run_large(const ClipArgs& ca, hipStream_t st) {
  launch_all<P, R, 32, 128, 64, RECHECK>(ca, false, st);
  VT_HIP(hipGetLastError());
  return VOTESS_OK;
}

}  // namespace

votess_status launch_clip(const ClipLaunch& a, hipStream_t st) {
  if (a.nc == 0) return VOTESS_OK;
  ClipArgs c;
  c.rec = a.sorted;
  c.n = a.n;
  c.lo0 = a.lo[0]; c.lo1 = a.lo[1]; c.lo2 = a.lo[2];
  c.hi0 = a.hi[0]; c.hi1 = a.hi[1]; c.hi2 = a.hi[2];
  c.cells = a.cells;
  c.nc = a.nc;
  c.knn = a.knn;
  c.k = a.k;
  c.kstride = a.knn_stride > 0 ? a.knn_stride : a.k;
  c.knn_by_id = a.knn_by_id;
  c.eps = a.eps;
  // k-lists ordered by float distances may misplace near-ties by a few ulp:
  // certify only with that much slack
  c.dmargin = a.knn_dist == VOTESS_F32 ? (1.0 - 8.0 * (double)FLT_EPSILON) : 1.0;
  c.max_nbr = a.max_nbr;
  c.max_vert = a.max_vert;
  c.out_by_id = a.out_by_id;
  c.status = a.status;
  c.nbr_count = a.nbr_count;
  c.nbr = a.nbr;
  c.volume = a.volume;
  c.kneeded = a.kneeded;
  c.vcount = a.vcount;
  c.verts = a.verts;
  c.vplanes = a.vplanes;
  c.area = a.area;
  c.centroid = a.centroid;
  c.r2out = a.r2out;
  c.counters = a.counters;
  for (int i = 0; i < kLevels; ++i) c.level[i] = a.level[i];
  c.stream = a.stream;
  c.cell_start = a.cell_start;
  c.grid = a.grid;
  c.sub = a.sub;
  const bool f32 = a.precision == VOTESS_CLIP_F32_RECHECK;
  if (f32 && a.dtype != VOTESS_F32) return fail(VOTESS_EINVAL, "clip: F32_RECHECK needs F32 positions");
  if (a.stream && (a.knn_dist == VOTESS_F32) != f32)
    return fail(VOTESS_EINVAL, "clip: the stream phase needs k-lists built in the clip precision");
  if (a.stream && !a.cell_start) return fail(VOTESS_EINVAL, "clip: the stream phase needs cell_start");
  c.rest = c.mark = c.save = 0;
  if (a.capacity == 0) {
    // in two launches, unless there is no list, two cells may share a row, or the
    // stream phase follows and the neighbour rows are the caller's (those of
    // uncertified cells are not to be written) or too short for a cell's state:
    // then one kernel does both, sooner than a second one that starts its cells
    // from the box again (2^20 clustered points, lists of 64: float 21.1 and 24.2
    // ms, double 23.3 and 27.2)
    const bool split =
        a.k > 0 && a.own_rows && (!a.stream || (a.spare_rows && a.max_nbr >= kStateWords));
    if (f32) return run_fast<float, float, true>(c, split, st);
    if (a.dtype == VOTESS_F32) return run_fast<float, double, false>(c, split, st);
    return run_fast<double, double, false>(c, split, st);
  }
  if (f32) return run_large<float, float, true>(c, st);
  if (a.dtype == VOTESS_F32) return run_large<float, double, false>(c, st);
  return run_large<double, double, false>(c, st);
}

}  // namespace votess

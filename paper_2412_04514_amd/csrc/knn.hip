// k-nearest-neighbour search over the grid (paper, Summary section: the
// neighbour search that follows the grid sort).
//
// A group of G lanes serves one query (queries in grid-sorted order, so that
// neighbouring groups scan overlapping grid cells), in two phases:
//   A. a seed block around the query -- sub-cells of its own dense cell, or
//      grid cells -- grown ring by ring until the cell / sub-cell starts show
//      at least K other points in it, then scanned whole: the list is full;
//   B. every other grid-cell row, and sub-cell row of a dense cell, that
//      meets the ball of the list's current K-th distance, each row cut to
//      the ball (which shrinks as the list improves): one contiguous range of
//      sorted points per row, split at dense cells.
// The control flow is the same in every lane of the group.  Rows are cut and
// looked up G at a time, one per lane; the candidates of the ranges found are
// taken G at a time, and each that beats the current K-th is gathered in LDS.
// G gathered ones are merged into the ascending list, which the group holds as
// E consecutive entries per lane, by one bitonic network.
// What bounds it: vector instructions (VALU 100% busy).  With the rows of phase
// B stepped through one by one by the whole group, in double, and candidates
// inserted one by one (~40 instructions for each of ~80 per query at k = 64),
// 64-lists took 4.36 ms for 2^20 uniform points in float, 22.8 ms for 4M
// clustered ones and 25.5 ms for 3M clustered ones in double; now 1.95, 14.7
// and 14.8 ms.
#include "internal.h"
#include "device_common.h"

#include <climits>

namespace votess {
namespace {

// List keys ordered by (d^2, sorted index).  FP32 distances pack into one
// u64: the bits of a non-negative float order like the float.
template <typename D>
struct KeyOps;
template <>
struct KeyOps<float> {
  using Key = unsigned long long;
  __device__ static Key make(float d2, int j) { return ((unsigned long long)__float_as_uint(d2) << 32) | (unsigned)j; }
  __device__ static Key inf() { return ~0ull; }
  __device__ static bool less(Key a, Key b) { return a < b; }
  __device__ static bool finite(Key a) { return a != ~0ull; }
  __device__ static double d2(Key a) { return (double)__uint_as_float((unsigned)(a >> 32)); }
  __device__ static int idx(Key a) { return a == ~0ull ? -1 : (int)(unsigned)(a & 0xffffffffu); }
  __device__ static Key pick(bool c, Key a, Key b) { return c ? a : b; }
  // f applied to each 32-bit word of the key
  template <class F>
  __device__ static Key each_word(Key a, F f) {
    return ((unsigned long long)f((unsigned)(a >> 32)) << 32) | f((unsigned)a);
  }
};
template <>
struct KeyOps<double> {
  struct Key {
    double d;
    int i;
  };
  __device__ static Key make(double d2, int j) { return {d2, j}; }
  // (above every point's key, the infinite d^2 of points too far apart included)
  __device__ static Key inf() { return {__builtin_inf(), INT_MAX}; }
  __device__ static bool less(Key a, Key b) { return a.d < b.d || (a.d == b.d && a.i < b.i); }
  __device__ static bool finite(Key a) { return a.i != INT_MAX; }
  __device__ static double d2(Key a) { return a.d; }
  __device__ static int idx(Key a) { return a.i == INT_MAX ? -1 : a.i; }
  // field by field: a choice between two structs as lvalues would select
  // their addresses and keep the list in scratch memory
  __device__ static Key pick(bool c, Key a, Key b) { return {c ? a.d : b.d, c ? a.i : b.i}; }
  template <class F>
  __device__ static Key each_word(Key a, F f) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(a.d);
    const unsigned long long w = ((unsigned long long)f((unsigned)(u >> 32)) << 32) | f((unsigned)u);
    return {__longlong_as_double((long long)w), (int)f((unsigned)a.i)};
  }
};

// Moves of 32-bit words between the lanes of a group of G consecutive lanes.
// For G = 8 or 16 they are DPP row operations, which stay in the vector
// ALU (controls: quad_perm [1,0,3,2] = 0xB1 takes lane ^ 1, [2,3,0,1] = 0x4E
// lane ^ 2, [3,2,1,0] = 0x1B reverses a quad, [3,3,3,3] = 0xFF broadcasts
// its last lane; row_mirror = 0x140 takes lane 15 - i within the row, row_half_mirror =
// 0x141 lane 7 - i within each eight); a group of 32 uses the LDS permute.
// Every lane of the group is active.
template <int CTRL>
__device__ __forceinline__ unsigned dpp_mov(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int G>
struct LaneMove {
  static_assert(G == 8 || G == 16 || G == 32, "the groups that have kernels");
  static constexpr bool kDpp = G <= 16;
  // the word of lane l ^ m (m a power of two below G)
  __device__ static unsigned xor_(unsigned v, int m) {
    if constexpr (kDpp) {
      if (m == 1) return dpp_mov<0xB1>(v);
      if (m == 2) return dpp_mov<0x4E>(v);
      if (m == 4) return dpp_mov<0x141>(dpp_mov<0x1B>(v));  // i -> 3 - i in the quad, then 7 - i
      if (m == 8) return dpp_mov<0x140>(dpp_mov<0x141>(v));  // 7 - i in the eight, then 15 - i
    }
    return (unsigned)__shfl_xor((int)v, m, 64);
  }
  // the word of the group's last lane
  __device__ static unsigned last(unsigned v, int gb, int l) {
    if constexpr (G == 8) {
      const unsigned a = dpp_mov<0xFF>(v);  // each quad: its last lane
      const unsigned b = dpp_mov<0x141>(a);  // the other quad's
      return l < 4 ? b : a;
    } else if constexpr (G == 16) {
      const unsigned a = dpp_mov<0xFF>(v), b = dpp_mov<0x140>(a), c = dpp_mov<0x141>(a), d = dpp_mov<0x140>(c);
      return l < 4 ? b : (l < 8 ? d : (l < 12 ? c : a));
    } else {
      return (unsigned)__shfl((int)v, gb + G - 1, 64);
    }
  }
};

// Ascending list of K keys over a group of G lanes: lane l holds ranks
// l E .. l E + E - 1.  Every call is made by all G lanes of the group.
template <typename D, int G, int E>
struct GroupList {
  using O = KeyOps<D>;
  using Key = typename O::Key;
  Key key[E];
  __device__ void init() {
#pragma unroll
    for (int e = 0; e < E; ++e) key[e] = O::inf();
  }
  using LM = LaneMove<G>;
  // the key of rank K0 - 1 (K0 a multiple of E)
  template <int K0>
  __device__ Key at(int gb, int l) const {
    static_assert(K0 % E == 0 && K0 <= G * E, "a lane's last key");
    return O::each_word(key[E - 1], [&](unsigned w) {
      if constexpr (K0 == G * E) return LM::last(w, gb, l);
      else return (unsigned)__shfl((int)w, gb + K0 / E - 1, 64);
    });
  }
  // Compare-exchange of positions i = l N + e and i ^ js over the G N keys
  // that the group holds N per lane: inside a lane in registers, across lanes
  // by lane moves; up(i) tells whether the pair is put in ascending order.
  template <int N, class F>
  __device__ __forceinline__ static void exchange(Key (&a)[N], int l, int js, F up) {
    if (js < N) {
#pragma unroll
      for (int e = 0; e < N; ++e) {
        const int pe = e ^ js;
        if (pe > e) {
          const Key x = a[e], y = a[pe];
          const bool sw = up(l * N + e) ? O::less(y, x) : O::less(x, y);
          a[e] = O::pick(sw, y, x);
          a[pe] = O::pick(sw, x, y);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) {
        const int i = l * N + e;
        const Key o = O::each_word(a[e], [&](unsigned w) { return LM::xor_(w, js / N); });
        const bool keep_min = up(i) == ((i & js) == 0);
        a[e] = O::pick(keep_min == O::less(o, a[e]), o, a[e]);
      }
    }
  }
  // Sorts G N keys ascending (G and N powers of two): a bitonic network.
  template <int N>
  __device__ __forceinline__ static void sort(Key (&a)[N], int l) {
#pragma unroll
    for (int ks = 2; ks <= G * N; ks <<= 1) {
#pragma unroll
      for (int js = ks >> 1; js > 0; js >>= 1) exchange<N>(a, l, js, [&](int i) { return (i & ks) == 0; });
    }
  }
  // The K smallest of the list and of the n <= G new keys in buf (LDS, G
  // entries), as the list: the new keys are sorted, laid against the list in
  // reverse (the element-wise smaller ones are the K smallest and form a
  // bitonic sequence), and that sequence is merged.  Keys are distinct (the
  // index is part of the key), so the result is the same as inserting them
  // one by one.
  __device__ __forceinline__ void merge(Key* buf, int n, int l) {
    constexpr int K = G * E;
    const Key b = buf[l];
    Key a[1] = {O::pick(l < n, b, O::inf())};
    sort<1>(a, l);
    buf[l] = a[0];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int r = K - 1 - (l * E + e);
      if (r < G) {
        // (masked, so that the address is never formed from one below buf)
        const Key o = buf[r & (G - 1)];
        key[e] = O::pick(O::less(o, key[e]), o, key[e]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
    for (int js = K / 2; js > 0; js >>= 1) exchange<E>(key, l, js, [](int) { return true; });
  }
};

// Held to 7 waves per SIMD with float keys and 6 with double ones, spills and
// all: at k = 64 on clustered input one wave less leaves latencies open and one
// more spills more (4M points, float: 15.1, 14.7 and 15.5 ms at 6, 7 and 8; 3M
// points, double: 15.2, 14.8 and 16.1 ms at 5, 6 and 7).
// Blocks are taken in an XCD-aware order: the hardware deals launched
// blocks round-robin over the eight XCDs, so launched block b runs logical
// block (b mod 8) per + b / 8 (per = blocks / 8, rounded up; the launch is
// padded to 8 per) and each XCD works on one contiguous stretch of the
// grid-sorted queries, whose candidates its own L2 then holds.
// The list holds LIST entries, of which the first K are asked for and bound the
// search.
template <typename T, typename D, int K, int LIST, int GS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(D) == 4 ? 7 : 6))) void k_knn(const typename Rec<T>::type* __restrict__ rec, int n, GridDev G,
                                             const int* __restrict__ cell_start, SubGrid sub,
                                             const int* __restrict__ queries, int nq, int* __restrict__ knn,
                                             unsigned* __restrict__ err, int nblocks) {
  constexpr int E = LIST / GS;
  static_assert(E * GS == LIST && K <= LIST, "LIST must be a multiple of GS, and hold K");
  using O = KeyOps<D>;
  using Key = typename O::Key;
  const int per = (nblocks + 7) / 8;
  const int lb = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
  if (lb >= nblocks) return;
  const int lane = threadIdx.x & 63;
  const int l = lane & (GS - 1), gb = lane - l;
  const int q = (int)(((long long)lb * blockDim.x + threadIdx.x) / GS);
  if (q >= nq) return;  // whole groups leave together
  const int s = queries ? queries[q] : q;
  const auto pr = rec[s];
  const D px = (D)pr.x, py = (D)pr.y, pz = (D)pr.z;
  const int cx = axis_cell((double)pr.x, G.lo0, G.ih0, G.g0);
  const int cy = axis_cell((double)pr.y, G.lo1, G.ih1, G.g1);
  const int cz = axis_cell((double)pr.z, G.lo2, G.ih2, G.g2);
  const double ext = fmax(G.hi0 - G.lo0, fmax(G.hi1 - G.lo1, G.hi2 - G.lo2));
  const double margin = 1e-9 * ext;  // covers floor() rounding at cell borders

  GroupList<D, GS, E> L;
  L.init();
  Key wk = O::inf();  // the list's k-th key (group-uniform)
  // Candidates that beat the K-th are gathered in LDS (per group) and merged
  // into the list GS at a time.
  constexpr int BUF = 2 * GS;
  __shared__ Key sbuf[(256 / GS) * BUF];
  Key* gbuf = sbuf + ((threadIdx.x & 255) / GS) * BUF;
  // point ranges being scanned, per group (two per lane at most)
  __shared__ int2 srng[(256 / GS) * 2 * GS];
  int2* grng = srng + ((threadIdx.x & 255) / GS) * 2 * GS;
  // row pieces that have to be walked cell by cell (x0, x1, y, z), per group
  __shared__ int4 swalk[(256 / GS) * 2 * GS];
  int4* gwalk = swalk + ((threadIdx.x & 255) / GS) * 2 * GS;
  // the group's place in the enumeration: the same for all its lanes, and held
  // here rather than in registers
  struct Place {
    int bx0, bx1, by0, by1, bz0, bz1;  // the seed block: sub-cells of the own cell, or grid cells
    int pb, np, ny, y0, z0;            // rows: next ordinal, their count, rows per layer, first row
    int wn, wp, x, x1, y, z;           // walks: listed, next one; the one being walked
    int dpb, dnp, dny, dy0, dz0, dcell;  // the dense cell's sub-rows, as above; the cell
  };
  __shared__ Place splace[256 / GS];
  Place& E_ = splace[(threadIdx.x & 255) / GS];
  int nbuf = 0;
  const double p0 = (double)pr.x, p1 = (double)pr.y, p2 = (double)pr.z;
  const unsigned long long gmask = (1ull << GS) - 1ull;
  const unsigned long long below = (1ull << l) - 1ull;
  auto gballot = [&](bool v) -> unsigned long long { return (__ballot(v) >> gb) & gmask; };

  // number of points in the rows of the seed block, summed over the group's lanes
  auto count_rows = [&](auto row_range) -> int {
    const int ny = E_.by1 - E_.by0 + 1, npairs = ny * (E_.bz1 - E_.bz0 + 1);
    int cnt = 0;
    for (int pi = l; pi < npairs; pi += GS) {
      const int kz = pi / ny;
      const int2 rg = row_range(E_.by0 + pi - kz * ny, E_.bz0 + kz);
      cnt += rg.y - rg.x;
    }
#pragma unroll
    for (int o = 1; o < GS; o <<= 1) cnt += __shfl_xor(cnt, o, 64);
    return cnt;
  };
  // squared search radius: the k-th distance with slack for float rounding
  // of d^2 (once the list is full)
  auto rad2 = [&]() { return O::d2(wk) * (1.0 + 1e-6); };
  // distance from p to [a, b], less the rounding margin
  auto gap = [&](double p, double a_, double b_) { return fmax(0.0, fmax(a_ - p, p - b_) - margin); };

  // ---- phase A: a seed block around the query that holds at least K other
  // points (counted from the cell and sub-cell starts), scanned whole; it
  // fills the list, and its k-th distance bounds the search
  const int c0 = cx + G.g0 * (cy + G.g1 * cz);
  const int2 info0 = sub.info ? sub.info[c0] : make_int2(-1, 0);
  const bool seed_sub = is_dense(info0) && cell_start[c0 + 1] - cell_start[c0] >= K + 1;
  int qx = cx, qy = cy, qz = cz, m0 = G.g0, m1 = G.g1, m2 = G.g2, base0 = 0;
  const int* srec = cell_start;  // row starts: grid cells, or the own cell's sub-cells
  if (seed_sub) {
    const SubCell sc = sub_cell(sub_record(sub, info0));
    srec = sc.start;
    base0 = cell_start[c0];
    m0 = sc.m0;
    m1 = sc.m1;
    m2 = sc.m2;
    qx = sub_axis(p0, sc.lo0, sc.ih0, m0);
    qy = sub_axis(p1, sc.lo1, sc.ih1, m1);
    qz = sub_axis(p2, sc.lo2, sc.ih2, m2);
  }
  auto seed_row = [&](int y, int z) -> int2 {
    const int row = m0 * (y + m1 * z);
    return make_int2(base0 + srec[row + E_.bx0], base0 + srec[row + E_.bx1 + 1]);
  };
  for (int r = 0;; ++r) {
    E_.bx0 = max(qx - r, 0); E_.bx1 = min(qx + r, m0 - 1);
    E_.by0 = max(qy - r, 0); E_.by1 = min(qy + r, m1 - 1);
    E_.bz0 = max(qz - r, 0); E_.bz1 = min(qz + r, m2 - 1);
    if (count_rows(seed_row) >= K + 1 || (E_.bx0 == 0 && E_.by0 == 0 && E_.bz0 == 0 && E_.bx1 == m0 - 1 &&
                                          E_.by1 == m1 - 1 && E_.bz1 == m2 - 1))
      break;
  }
  // Its rows go outward from the query's (offsets 0, +1, -1, +2, ... in z, and
  // in y within each z), so that the list's first K candidates lie near the
  // query and fewer later ones displace them.
  E_.pb = 0;
  E_.ny = 2 * max(qy - E_.by0, E_.by1 - qy) + 1;
  E_.np = E_.ny * (2 * max(qz - E_.bz0, E_.bz1 - qz) + 1);

  // ---- The search.  One loop alternates between scanning what is listed, GS
  // candidates at a time (a batch takes the rest of one range and the start of
  // the next ones), and listing the next ranges, GS rows at a time, one per
  // lane.  (One loop, so that the scan and the merge exist once: as functions
  // of their own they would reach the group's LDS through generic pointers.)
  // Phase A lists the seed block's rows.  Phase B lists every other grid row
  // and sub-row that meets the ball of the k-th distance, cut to the ball
  // (which shrinks as the list improves).
  enum { kSeed, kSquare, kRows, kWalk, kDense, kDone };
  int stage = kSeed;
  bool drain = false;  // merge whatever is gathered before going on
  int rn = 0, rp = 0, cur = 0, end = 0;
  for (;;) {
    if (nbuf >= GS || (drain && nbuf > 0)) {
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      const int take = min(nbuf, GS), left = nbuf - take;
      const Key rest = gbuf[GS + l];  // (read before the merge uses the buffer)
      L.merge(gbuf, take, l);
      if (l < left) gbuf[l] = rest;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      nbuf = left;
      wk = L.template at<K>(gb, l);
      if (drain) continue;
    }
    drain = false;
    if (cur < end || rp < rn) {  // a batch of candidates
      int jj = -1, nb = 0;
      for (;;) {
        const int take = min(GS - nb, end - cur);
        if (l >= nb && l < nb + take) jj = cur + (l - nb);
        nb += take;
        cur += take;
        if (nb == GS || rp >= rn) break;
        const int2 rg = grng[rp];
        ++rp;
        cur = rg.x;
        end = rg.y;
      }
      Key ck = O::inf();
      const bool valid = jj >= 0 && jj != s;
      if (valid) {
        const auto qr = rec[jj];
        ck = O::make(dist2_nc((D)qr.x - px, (D)qr.y - py, (D)qr.z - pz), jj);
      }
      const bool pass = valid && O::less(ck, wk);
      const unsigned long long m = gballot(pass);
      if (pass) gbuf[nbuf + __popcll(m & below)] = ck;
      nbuf += __popcll(m);
      continue;
    }
    if (stage == kDone) break;
    int2 ra = make_int2(0, 0), rb = make_int2(0, 0);  // this lane's ranges
    if (stage == kSeed) {
      const int pi = E_.pb + l;
      if (pi < E_.np) {
        const int kz = pi / E_.ny, ky = pi - kz * E_.ny;
        const int z = qz + ((kz & 1) ? (kz + 1) >> 1 : -(kz >> 1));
        const int y = qy + ((ky & 1) ? (ky + 1) >> 1 : -(ky >> 1));
        if (z >= E_.bz0 && z <= E_.bz1 && y >= E_.by0 && y <= E_.by1) ra = seed_row(y, z);
      }
      E_.pb += GS;
      if (E_.pb >= E_.np) {
        stage = kSquare;
      }
    } else if (stage == kSquare) {
      if (nbuf > 0) {  // the seed block's K-th first
        drain = true;
        continue;
      }
      stage = kDone;
      if (O::finite(wk)) {
        const double r0 = sqrt(rad2()) + margin;
        const int gz0 = axis_cell(p2 - r0, G.lo2, G.ih2, G.g2), gz1 = axis_cell(p2 + r0, G.lo2, G.ih2, G.g2);
        const int gy0 = axis_cell(p1 - r0, G.lo1, G.ih1, G.g1), gy1 = axis_cell(p1 + r0, G.lo1, G.ih1, G.g1);
        const int gx0 = axis_cell(p0 - r0, G.lo0, G.ih0, G.g0), gx1 = axis_cell(p0 + r0, G.lo0, G.ih0, G.g0);
        // (a ball inside a seed block of grid cells has been scanned)
        if (seed_sub || gx0 < E_.bx0 || gx1 > E_.bx1 || gy0 < E_.by0 || gy1 > E_.by1 || gz0 < E_.bz0 ||
            gz1 > E_.bz1) {
          E_.pb = 0;
          E_.ny = gy1 - gy0 + 1;
          E_.np = E_.ny * (gz1 - gz0 + 1);
          E_.y0 = gy0;
          E_.z0 = gz0;
          E_.wn = E_.wp = 0;
          stage = kRows;
        }
      }
      continue;
    } else if (stage == kRows) {
      if (E_.wp < E_.wn) {
        // a listed piece, cut again to the ball as it is now
        const int4 w = gwalk[E_.wp];
        ++E_.wp;
        const double gz = gap(p2, G.lo2 + w.w * G.h2, G.lo2 + (w.w + 1) * G.h2);
        const double gy = gap(p1, G.lo1 + w.z * G.h1, G.lo1 + (w.z + 1) * G.h1);
        const double rem = rad2() - gz * gz - gy * gy;
        if (rem >= 0.0) {
          const double rx = sqrt(rem) + margin;
          E_.x = max(w.x, axis_cell(p0 - rx, G.lo0, G.ih0, G.g0));
          E_.x1 = min(w.y, axis_cell(p0 + rx, G.lo0, G.ih0, G.g0));
          E_.y = w.z;
          E_.z = w.w;
          stage = kWalk;
        }
        continue;
      }
      if (E_.pb >= E_.np) {
        stage = kDone;
        drain = true;
        continue;
      }
      // the next rows of the square: each lane cuts its row to the ball,
      // leaves out the seed block's cells (scanned whole) and reads what is
      // left, at most one piece on either side.  Pieces of at most kSubMin
      // points hold no dense cell and are scanned together; the others are
      // walked one by one.
      const int pi = E_.pb + l;
      E_.pb += GS;
      int xa0 = 1, xa1 = 0, xb0 = 1, xb1 = 0, y = 0, z = 0;
      if (pi < E_.np) {
        const int kz = pi / E_.ny;
        z = E_.z0 + kz;
        y = E_.y0 + (pi - kz * E_.ny);
        const double gz = gap(p2, G.lo2 + z * G.h2, G.lo2 + (z + 1) * G.h2);
        const double gy = gap(p1, G.lo1 + y * G.h1, G.lo1 + (y + 1) * G.h1);
        const double rem = rad2() - gz * gz - gy * gy;
        if (rem >= 0.0) {
          const double rx = sqrt(rem) + margin;
          xa0 = axis_cell(p0 - rx, G.lo0, G.ih0, G.g0);
          xa1 = axis_cell(p0 + rx, G.lo0, G.ih0, G.g0);
          if (!seed_sub && y >= E_.by0 && y <= E_.by1 && z >= E_.bz0 && z <= E_.bz1) {
            xb0 = max(xa0, E_.bx1 + 1);
            xb1 = xa1;
            xa1 = min(xa1, E_.bx0 - 1);
          }
          const int row = G.g0 * (y + G.g1 * z);
          if (xa0 <= xa1) ra = make_int2(cell_start[row + xa0], cell_start[row + xa1 + 1]);
          if (xb0 <= xb1) rb = make_int2(cell_start[row + xb0], cell_start[row + xb1 + 1]);
        }
      }
      const bool wa = ra.y - ra.x > kSubMin, wb = rb.y - rb.x > kSubMin;
      const unsigned long long ma = gballot(wa), mb = gballot(wb);
      if (ma | mb) {
        const int w = __popcll(ma & below) + __popcll(mb & below);
        if (wa) {
          gwalk[w] = make_int4(xa0, xa1, y, z);
          ra = make_int2(0, 0);
        }
        if (wb) {
          gwalk[w + (wa ? 1 : 0)] = make_int4(xb0, xb1, y, z);
          rb = make_int2(0, 0);
        }
      }
      E_.wn = __popcll(ma) + __popcll(mb);
      E_.wp = 0;
    } else if (stage == kWalk) {
      if (E_.x > E_.x1) {
        stage = kRows;
        continue;
      }
      // the stretch of cells without sub-grids: the group reads GS
      // consecutive cells' records at once and ends it at the first dense one
      const int row = G.g0 * (E_.y + G.g1 * E_.z), x = E_.x, x1 = E_.x1;
      int xe = x;
      for (;;) {
        const int xc = xe + l;
        const bool dense = xc <= x1 && sub.info && is_dense(sub.info[row + xc]);
        const unsigned long long dm = gballot(dense);
        if (dm) {
          xe += __ffsll((long long)dm) - 1;
          break;
        }
        xe += GS;
        if (xe > x1) {
          xe = x1 + 1;
          break;
        }
      }
      if (xe > x) {
        cur = cell_start[row + x];
        end = cell_start[row + xe];
        E_.x = xe;
        continue;
      }
      // dense cell: the square of its sub-rows that meets the ball
      const SubCell sc = sub_cell(sub_record(sub, sub.info[row + x]));
      const double r0 = sqrt(rad2()) + margin;
      const int sz0 = sub_axis(p2 - r0, sc.lo2, sc.ih2, sc.m2), sz1 = sub_axis(p2 + r0, sc.lo2, sc.ih2, sc.m2);
      const int sy0 = sub_axis(p1 - r0, sc.lo1, sc.ih1, sc.m1), sy1 = sub_axis(p1 + r0, sc.lo1, sc.ih1, sc.m1);
      E_.dpb = 0;
      E_.dny = sy1 - sy0 + 1;
      E_.dnp = E_.dny * (sz1 - sz0 + 1);
      E_.dy0 = sy0;
      E_.dz0 = sz0;
      E_.dcell = row + x;
      E_.x = x + 1;
      stage = kDense;
      continue;
    } else {  // kDense
      if (E_.dpb >= E_.dnp) {
        stage = kWalk;
        continue;
      }
      // the next sub-rows: each lane cuts its own to the ball, leaves out the
      // seed block's sub-cells and reads what is left
      const int c = E_.dcell;
      const SubCell sc = sub_cell(sub_record(sub, sub.info[c]));
      const int base = cell_start[c];
      const double w1 = 1.0 / sc.ih1, w2 = 1.0 / sc.ih2;
      const double ylo = G.lo1 + E_.y * G.h1, yhi = ylo + G.h1, zlo = G.lo2 + E_.z * G.h2, zhi = zlo + G.h2;
      const int pi = E_.dpb + l;
      E_.dpb += GS;
      if (pi < E_.dnp) {
        const int kz = pi / E_.dny;
        const int sz = E_.dz0 + kz, sy = E_.dy0 + (pi - kz * E_.dny);
        const double za = sz == 0 ? zlo : sc.lo2 + sz * w2, zb = sz == sc.m2 - 1 ? zhi : sc.lo2 + (sz + 1) * w2;
        const double ya = sy == 0 ? ylo : sc.lo1 + sy * w1, yb = sy == sc.m1 - 1 ? yhi : sc.lo1 + (sy + 1) * w1;
        const double gz = gap(p2, za, zb), gy = gap(p1, ya, yb);
        const double rem = rad2() - gz * gz - gy * gy;
        if (rem >= 0.0) {
          const double rx = sqrt(rem) + margin;
          int sx0 = sub_axis(p0 - rx, sc.lo0, sc.ih0, sc.m0);
          const int sx1 = sub_axis(p0 + rx, sc.lo0, sc.ih0, sc.m0);
          const int* st = sc.start + sc.m0 * (sy + sc.m1 * sz);
          if (seed_sub && c == c0 && sy >= E_.by0 && sy <= E_.by1 && sz >= E_.bz0 && sz <= E_.bz1) {
            if (sx0 < E_.bx0) ra = make_int2(base + st[sx0], base + st[min(sx1, E_.bx0 - 1) + 1]);
            sx0 = max(sx0, E_.bx1 + 1);
          }
          if (sx0 <= sx1) rb = make_int2(base + st[sx0], base + st[sx1 + 1]);
        }
      }
    }
    // list the ranges found, in lane order
    const bool ka = ra.x < ra.y, kb = rb.x < rb.y;
    const unsigned long long ba = gballot(ka), bb = gballot(kb);
    const int w = __popcll(ba & below) + __popcll(bb & below);
    if (ka) grng[w] = ra;
    if (kb) grng[w + (ka ? 1 : 0)] = rb;
    rn = __popcll(ba) + __popcll(bb);
    rp = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
  int* out = knn + (size_t)q * K;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (l * E + e < K) out[l * E + e] = O::idx(L.key[e]);
  if (l == 0 && O::finite(L.key[0]) && O::d2(L.key[0]) == 0.0) atomicOr(err, ERR_DUPLICATE);
}

template <typename T, typename D>
votess_status dispatch_k(int k, const void* sorted, int n, const GridDev& G, const int32_t* cs, const SubGrid& sub,
                         const int32_t* qs, int nq, int32_t* knn, unsigned* err, hipStream_t st) {
  using R4 = typename Rec<T>::type;
  const R4* rec = (const R4*)sorted;
  // A list is a power of two long, at least k; its first k entries are the
  // k-list, and the k-th bounds the search (1M clustered points, double, k = 24:
  // 2.81 ms, bounded by the 32nd 3.37).  (Merging needs a power of two, and beats
  // inserting by far: 2^20 uniform points, float, lists of 64 2.0 ms, lists of 48
  // by insertion 3.2 ms.)
#define VT_KNN_CASE(KK, LIST, GG)                                                                 \
  case KK: {                                                                                      \
    const int blocks = (int)(((long long)nq * GG + 255) / 256);                                   \
    const unsigned launched = (unsigned)(8 * ((blocks + 7) / 8));                                 \
    k_knn<T, D, KK, LIST, GG><<<launched, 256, 0, st>>>(rec, n, G, cs, sub, qs, nq, knn, err, blocks); \
    break;                                                                                        \
  }
  switch (k) {
    VT_KNN_CASE(8, 8, 8)
    VT_KNN_CASE(12, 16, 16)
    VT_KNN_CASE(16, 16, 16)
    VT_KNN_CASE(24, 32, 8)
    VT_KNN_CASE(32, 32, 8)
    VT_KNN_CASE(48, 64, 16)
    VT_KNN_CASE(64, 64, 16)
    VT_KNN_CASE(128, 128, 16)
    VT_KNN_CASE(256, 256, 32)
    default:
      return fail(VOTESS_EINVAL, "knn: k=%d has no kernel (k must be one of 8,12,16,24,32,48,64,128,256)", k);
  }
#undef VT_KNN_CASE
  VT_HIP(hipGetLastError());
  return VOTESS_OK;
}

}  // namespace

votess_status launch_knn(votess_ctx* ctx, const void* sorted, votess_dtype dt, int n, const GridDev& G,
                         const int32_t* cell_start, const SubGrid& sub, const int32_t* queries, int nq, int k,
                         votess_dtype dist, int32_t* knn, hipStream_t st) {
  if (nq == 0) return VOTESS_OK;
  if (dt == VOTESS_F64 && dist == VOTESS_F32)
    return fail(VOTESS_EINVAL, "knn: F32 distances need F32 positions");
  if (dt == VOTESS_F32) {
    if (dist == VOTESS_F32) return dispatch_k<float, float>(k, sorted, n, G, cell_start, sub, queries, nq, knn, ctx->d_err, st);
    return dispatch_k<float, double>(k, sorted, n, G, cell_start, sub, queries, nq, knn, ctx->d_err, st);
  }
  return dispatch_k<double, double>(k, sorted, n, G, cell_start, sub, queries, nq, knn, ctx->d_err, st);
}

}  // namespace votess

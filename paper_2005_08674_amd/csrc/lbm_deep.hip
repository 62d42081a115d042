// lbm_deep.hip -- several time steps per launch for a lattice with any edges
// (NSBC, periodic, velocity inlet): what lbm_step runs when no launch has been
// chosen for the lattice, as far as it is faster there than single steps and the
// 64-wide sweeps.
//
// A block owns a TX x TY output tile and computes it k <= KM steps ahead.  Its
// region is the tile widened by KM - 1 nodes on every side, one node per
// thread; level l (t + l) is needed on the tile widened by k - l, so the region
// shrinks by a ring per level and nothing is exchanged between blocks.  Level 1
// is pulled from memory, the others from LDS, in place: every thread reads its
// node's nine pulls, a barrier, every thread writes its collided node, a
// barrier.  Levels are held in the storage format, encoded as a store would
// write them, and every node runs the single-step path's operations in their
// order: results are bit-identical to single steps.
//
// The lattice's perimeter nodes inside the region (NSBC, velocity inlet, or
// periodic, which the single-step edge kernel also updates in decoded form) go to
// EW wavefronts of their own, packed into consecutive lanes, so that their
// longer chain runs beside the interior nodes' instead of in front of it.
//
// Why: a lattice of 128^2 keeps one step's launch busy for about 5.8 us, all of
// it latency (launch, the last-level cache's round trip, the NSBC chain); a
// level here costs LDS latency and arithmetic only.  A larger lattice gains the
// memory traffic of the steps in between, at the price of the margin.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm_device.h"
#include "lbm_launch.h"
#include "lbm_twostep_lds.h"

namespace lbm {

template <int TX, int TY, int KM>
struct DeepShape {
  static constexpr int W = TX + 2 * (KM - 1), H = TY + 2 * (KM - 1), N = W * H;
  static constexpr int NM = (N + 63) / 64 * 64;                 // threads of interior nodes
  static constexpr int EW = (2 * H + 2 * (W - 2) + 63) / 64;    // wavefronts of perimeter nodes
  static constexpr int NT = NM + 64 * EW;
};

// Register budget: two blocks of a wide shape on a CU for the 32-bit arithmetic
// (64 VGPRs for 32 x 16, 80 for 16 x 16; the perimeter path would take 93 and
// spills instead: 4096^2 FP32 162 -> 125 us a step, 512^2 with 16 x 16 tiles 5.0
// -> 3.7).  FP64 needs its 127-149 (16 x 16 held to 80: 256^2 2.6 -> 3.2).
template <int S, int NT>
constexpr int deep_waves() {
  return S == ST_F64 ? 1 : (NT == 1024 ? 8 : (NT == 704 ? 6 : 1));
}

template <int S, int CM, bool UB0, int TX, int TY, int KM>
__global__ __launch_bounds__((DeepShape<TX, TY, KM>::NT), (deep_waves<S, DeepShape<TX, TY, KM>::NT>())) void k_deep(LatDesc L, int parity, int tiles_x, int ntiles,
                                                                     int k) {
  using D = DeepShape<TX, TY, KM>;
  using C = Codec<S>;
  using T = typename C::T;
  using R = typename C::R;
  constexpr int W = D::W, H = D::H, N = D::N;
  __shared__ T lds[9 * N];
  // XCD x works through the x-th eighth of the row-major tiles: neighbouring
  // tiles, which share their margins, in one L2
  const int per = (ntiles + 7) >> 3, tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (tile >= ntiles) return;  // the whole block, before any barrier
  const int nx = L.nx, ny = L.ny, pitch = L.pitch;
  const int xo = tile % tiles_x * TX, yo = tile / tiles_x * TY;
  // every tile is whole: the last of a row or column moves back to end at the
  // lattice's, and stores only the nodes its neighbour does not
  const int x0 = min(xo, nx - TX), y0 = min(yo, ny - TY);
  const bool xper = L.bc[E_LEFT] == BC_PERIODIC, yper = L.bc[E_BOTTOM] == BC_PERIODIC;
  const int tid = threadIdx.x;
  const bool edge = __builtin_amdgcn_readfirstlane(tid) >= D::NM;  // the same for a whole wavefront

  // this thread's node: region position (cx, r), lattice position (x, y)
  int cx, r;
  bool act;
  if (!edge) {
    r = tid / W;
    cx = tid - r * W;
    act = tid < N;
  } else {
    // perimeter columns and rows inside the region (at most one of each side):
    // the columns' nodes first, then the rows' others
    auto at = [](int p, int o, int n, int len) {  // region coordinate of lattice coordinate p (mod n), or -1
      int q = p - o;
      if (q >= n) q -= n;
      return q >= 0 && q < len ? q : (q + n < len ? q + n : -1);
    };
    const int ox = x0 - (KM - 1), oy = y0 - (KM - 1);
    const int ca = at(0, ox, nx, W), cb = at(nx - 1, ox, nx, W), ra = at(0, oy, ny, H), rb = at(ny - 1, oy, ny, H);
    const int nc = (ca >= 0) + (cb >= 0), nr = (ra >= 0) + (rb >= 0);
    const int c1 = nc == 2 ? min(ca, cb) : max(ca, cb), c2 = nc == 2 ? max(ca, cb) : W;
    int e = tid - D::NM;
    if (e < nc * H) {
      cx = e < H ? c1 : c2;
      r = e < H ? e : e - H;
      act = true;
    } else {
      e -= nc * H;
      const int len = W - nc;
      const bool first = e < len;
      act = e < nr * len;
      cx = first ? e : e - len;
      if (nc > 0 && cx >= c1) ++cx;
      if (nc == 2 && cx >= c2) ++cx;
      r = first ? (ra >= 0 ? ra : rb) : rb;
    }
  }
  int x = x0 - (KM - 1) + cx, y = y0 - (KM - 1) + r;
  if (xper) x += x < 0 ? nx : (x >= nx ? -nx : 0);
  if (yper) y += y < 0 ? ny : (y >= ny ? -ny : 0);
  const bool perimeter = x == 0 || x == nx - 1 || y == 0 || y == ny - 1;
  act = act && x >= 0 && x < nx && y >= 0 && y < ny && perimeter == edge;
  // the last level the node is needed at
  const int depth = min(min(cx, W - 1 - cx), min(r, H - 1 - r));
  const int last = act ? depth - (KM - 1) + k : 0;
  const bool stores = last >= k && x >= xo && y >= yo;

  const T* __restrict__ A = static_cast<const T*>(buf_of(L, parity));
  const int64_t plane = L.plane;
  const R rho0 = R(L.rho0), omega = R(L.omega);
  Base<R> base(L);
  base.zero = UB0;
  const OutPlanes<T> out(static_cast<T*>(buf_of(L, parity ^ 1)), plane);
  const uint32_t own = (uint32_t)(y * pitch + x) * (uint32_t)sizeof(T);
  T* const node = lds + (r * W + cx);
  // a level's values v of this node: to LDS, or the last level's to memory
  auto keep = [&](int l, const T v[9]) __attribute__((always_inline)) {
    if (l < k) {
#pragma unroll
      for (int i = 0; i < 9; ++i) node[i * N] = v[i];
    } else if (stores) {
#pragma unroll
      for (int i = 0; i < 9; ++i) out.template put<false>(i, own, v[i]);
    }
  };
  // Both kinds of wavefront pass the same barriers: one after a level's writes
  // (but the last's), one after its reads (but the first's).
  R g[9];
  if (!edge) {
    // not on the perimeter: no pull wraps or leaves the lattice
    auto update = [&](int l) __attribute__((always_inline)) {
      collide_stored<S, CM>(L, g, rho0, base, omega);
      T v[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) v[i] = C::raw_enc(g[i]);
      keep(l, v);
    };
    if (last >= 1) {
      const uint32_t row = (uint32_t)pitch * (uint32_t)sizeof(T);
      const uint32_t ro[3] = {own + row, own, own - row};
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = C::raw(ldg(A + i * plane, ro[1 + kCy[i]] - kCx[i] * (int)sizeof(T)));
      update(1);
    }
    if (k > 1) __syncthreads();
    for (int l = 2; l <= k; ++l) {
      if (l <= last) {
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = C::raw(node[i * N - kCy[i] * W - kCx[i]]);
      }
      __syncthreads();
      if (l <= last) update(l);
      if (l < k) __syncthreads();
    }
    return;
  }

  // Perimeter nodes.  (dx, dy): inward directions of the NSBC edges the node is on
  // (0: none).
  const int bl = x == 0 ? L.bc[E_LEFT] : (x == nx - 1 ? L.bc[E_RIGHT] : (int)BC_PERIODIC);
  const int bb = y == 0 ? L.bc[E_BOTTOM] : (y == ny - 1 ? L.bc[E_TOP] : (int)BC_PERIODIC);
  const int dx = bl == BC_NSBC ? (x == 0 ? 1 : -1) : 0, dy = bb == BC_NSBC ? (y == 0 ? 1 : -1) : 0;
  const int vel = bl == BC_VELOCITY ? (x == 0 ? -1 : 1) : 0;
  const uint32_t unknown = tl_unknown(xper ? 1 : x, yper ? 1 : y, xper ? 3 : nx, yper ? 3 : ny);
  // A level's update from `pull(px, py, i)`, population i of the node (px, py)
  // away (within one of it; an unknown one is read at the nearest node of the
  // lattice and dropped), and `mom(px, py, m)`, the moments of the node itself or
  // of one up to two nodes inward of an NSBC edge.  Those lie in the region and are
  // there at the level before: an NSBC edge crosses a region only as an outermost
  // row or column of the tile (tiles are whole and a margin narrower than a tile,
  // deep_supported), so two nodes inward is a row or column of the tile, no nearer
  // to the region's border than the node.
  static_assert(TX >= 3 && TY >= 3, "NSBC reads two nodes inward");
  const int xm = x == 0 && !xper ? 0 : -1, xp = x == nx - 1 && !xper ? 0 : 1;
  const int ym = y == 0 && !yper ? 0 : -1, yp = y == ny - 1 && !yper ? 0 : 1;
  M3<R> mc = {{R(0), R(0), R(0)}};
  auto gather = [&](auto pull, auto mom) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const R v = C::dec(pull(kCx[i] > 0 ? xm : (kCx[i] < 0 ? xp : 0), kCy[i] > 0 ? ym : (kCy[i] < 0 ? yp : 0), i), L.ds[i]);
      g[i] = (unknown >> i) & 1u ? R(0) : v;
    }
    if (dx | dy) mc = predict_at<R>(L, dx, dy, mom);
  };
  auto update = [&](int l) __attribute__((always_inline)) {
    if (vel)
      mc = velocity_edge_moments<R>(g, vel, rho0, in_type<R>(L.uw[0], L.uwf[0]), in_type<R>(L.duw[0], L.duwf[0]),
                                    in_type<R>(L.duw[1], L.duwf[1]));
    if (unknown) nsbc_assign_correct<R>(g, unknown, mc, rho0, base, L.corr_mode);
    collide<R, CM>(L, g, rho0, base, omega);
    T v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) v[i] = C::enc(g[i], L.es[i]);
    keep(l, v);
  };
  if (last >= 1) {
    // a periodic side's neighbours lie across the lattice
    auto off = [&](int px, int py) {
      int sx = x + px, sy = y + py;
      if (xper) sx += sx < 0 ? nx : (sx >= nx ? -nx : 0);
      if (yper) sy += sy < 0 ? ny : (sy >= ny ? -ny : 0);
      return (uint32_t)(sy * pitch + sx) * (uint32_t)sizeof(T);
    };
    gather([&](int px, int py, int i) { return ldg(A + i * plane, off(px, py)); },
           [&](int px, int py, R m[3]) {
             R q[9];
             const uint32_t o = off(px, py);
#pragma unroll
             for (int i = 0; i < 9; ++i) q[i] = C::dec(ldg(A + i * plane, o), L.ds[i]);
             moments<R>(q, rho0, base, m[0], m[1], m[2]);
           });
    update(1);
  }
  if (k > 1) __syncthreads();
  for (int l = 2; l <= k; ++l) {
    if (l <= last)
      gather([&](int px, int py, int i) { return node[i * N + py * W + px]; },
             [&](int px, int py, R m[3]) {
               R q[9];
#pragma unroll
               for (int i = 0; i < 9; ++i) q[i] = C::dec(node[i * N + py * W + px], L.ds[i]);
               moments<R>(q, rho0, base, m[0], m[1], m[2]);
             });
    __syncthreads();
    if (l <= last) update(l);
    if (l < k) __syncthreads();
  }
}

// Tiles, and the largest number of steps, of the compiled shapes.
#define LBM_DEEP(X) \
  X(8, 8, 5)        \
  X(16, 16, 5)      \
  X(32, 16, 4)

struct DeepRow {
  int tx, ty, km;
};
static const DeepRow kDeep[] = {
#define X(a, b, c) {a, b, c},
    LBM_DEEP(X)
#undef X
};

int num_deep() { return sizeof(kDeep) / sizeof(kDeep[0]); }
int deep_steps(int id) { return kDeep[id].km; }
int64_t deep_tiles(const LatDesc& L, int id) {
  return (int64_t)((L.nx + kDeep[id].tx - 1) / kDeep[id].tx) * ((L.ny + kDeep[id].ty - 1) / kDeep[id].ty);
}
bool deep_supported(const LatDesc& L, int id) {
  // the region holds at most one perimeter column of each side and wraps at most once
  const int m = 2 * kDeep[id].km;
  return !(L.closure && L.net) && L.nx >= kDeep[id].tx + m && L.ny >= kDeep[id].ty + m;
}

template <int S, int TX, int TY, int KM>
static hipError_t launch_deep_t(const LatDesc& L, int parity, int k, hipStream_t s) {
  const int tx = (L.nx + TX - 1) / TX, n = tx * ((L.ny + TY - 1) / TY);
  const dim3 grid((n + 7) / 8 * 8), block(DeepShape<TX, TY, KM>::NT);
  auto launch = [&](auto cm, auto ub0) {
    k_deep<S, decltype(cm)::value, decltype(ub0)::value, TX, TY, KM><<<grid, block, 0, s>>>(L, parity, tx, n, k);
  };
  const std::integral_constant<int, COLL_MRT> mrt;
  const std::integral_constant<int, COLL_BGK> bgk;
  if (L.coll == COLL_MRT)
    L.ub_zero ? launch(mrt, std::true_type{}) : launch(mrt, std::false_type{});
  else
    L.ub_zero ? launch(bgk, std::true_type{}) : launch(bgk, std::false_type{});
  return hipGetLastError();
}

template <int S>
static hipError_t launch_deep_s(const LatDesc& L, int parity, int id, int k, hipStream_t s) {
  int n = 0;
#define X(a, b, c)                                                      \
  if (id == n) return launch_deep_t<S, a, b, c>(L, parity, k, s);      \
  ++n;
  LBM_DEEP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_deep(const LatDesc& L, int parity, int id, int k, hipStream_t s) {
  if (id < 0 || id >= num_deep() || k < 1 || k > kDeep[id].km || !deep_supported(L, id)) return hipErrorInvalidValue;
  switch (L.store) {
    case ST_F64: return launch_deep_s<ST_F64>(L, parity, id, k, s);
    case ST_F32: return launch_deep_s<ST_F32>(L, parity, id, k, s);
    case ST_F16: return launch_deep_s<ST_F16>(L, parity, id, k, s);
    case ST_BF16: return launch_deep_s<ST_BF16>(L, parity, id, k, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm

// lbm_twostep.hip -- the two-step sweep (t -> t + 2 in one launch, level
// t + 1 in LDS) and the three-step sweep (t -> t + 3, levels t + 1 and t + 2
// in LDS; lbm_twostep_lds.h) for lattices with NSBC on all four edges: their
// compile-time shapes, one instance per storage format and collision model,
// and their host-side launchers.
#include <hip/hip_runtime.h>

#include <vector>

#include <cstdio>

#include "lbm_device.h"
#include "lbm_launch.h"
#include "lbm_threestep.h"
#include "lbm_twostep_lds.h"

namespace lbm {

// ------------------------------------------------------------------ two-step kernel
// Candidate shapes of the two-step sweep (lbm_twostep_lds.h): output tile
// 64 x TY, NT threads per block, non-temporal stores (NTS), block -> tile map
// (MAP).  Workgroups go to the 8 XCDs round-robin (block b on XCD b mod 8),
// each XCD with its own L2, and a tile re-reads its neighbours' edge cache
// lines for its margin:
//   MAP 0: a 2-D grid, tile = (blockIdx.x, blockIdx.y); horizontal
//          neighbours run on different XCDs.
//   MAP 1: a 1-D grid over the row-major tiles in runs of 64 blocks; XCD k
//          takes 8 consecutive tiles of each run, so 7 of 8 horizontal
//          neighbours share an L2.
//   MAP 2: XCD k takes the k-th contiguous eighth of the row-major tiles, so
//          horizontal and vertical neighbours share an L2 except at the
//          eight band boundaries.
// TY and NT trade the margin's share of the work, the idle lanes of the last
// pass over the (TY + 2) x 68 and TY x 64 nodes, and the blocks that fit in
// a CU's LDS.
#define LBM_TWO_STEP(X)  \
  X(12, 512, true, 0)    \
  X(16, 512, true, 0)    \
  X(16, 512, true, 1)    \
  X(12, 512, true, 2)    \
  X(16, 512, true, 2)    \
  X(20, 512, true, 2)    \
  X(8, 256, true, 2)     \
  X(12, 384, true, 2)    \
  X(24, 768, true, 2)    \
  X(20, 768, true, 2)

template <int S, int TY, int NT, bool NTS, int CM, int MAP>
__global__ __launch_bounds__(NT, two_step_waves<S>()) void k_two_step(LatDesc L, int parity, int tiles_x,
                                                                    int tiles_y) {
  int txi, tyi;
  if (MAP == 0) {
    txi = blockIdx.x;
    tyi = blockIdx.y;
  } else {
    const int b = blockIdx.x, ntiles = tiles_x * tiles_y;
    int tile;
    if (MAP == 1) {
      tile = (b & ~63) + ((b & 7) << 3) + ((b >> 3) & 7);
    } else {
      const int per = (ntiles + 7) >> 3;
      tile = (b & 7) * per + (b >> 3);
    }
    if (tile >= ntiles) return;  // padding blocks: the whole block leaves before any barrier
    tyi = tile / tiles_x;
    txi = tile - tyi * tiles_x;
  }
  two_step_tile<S, TY, NT, NTS, CM>(L, parity, txi, tyi);
}

// the tile shapes first, then the marched ones (mr > 0: rows per round, h:
// chunk rows)
struct TwoStepShape {
  int ty, nt;
  bool nts;
  int map, mr, h;
};
static const TwoStepShape kTwo[] = {
#define X(a, b, c, d) {a, b, c, d, 0, 0},
    LBM_TWO_STEP(X)
#undef X
#define X(a, m, b, h, n) {a, b, n, 2, m, h},
    LBM_TWO_MARCH(X)
#undef X
};
static constexpr int kNumTwo = sizeof(kTwo) / sizeof(kTwo[0]);
static constexpr int kNumTwoMarch = 0
#define X(a, m, b, h, n) +1
    LBM_TWO_MARCH(X)
#undef X
    ;

bool two_step_is_march(int id) { return id >= 0 && id < kNumTwo && kTwo[id].mr > 0; }

int num_two_step() { return kNumTwo; }

void two_step_name(int id, char* buf, size_t len) {
  if (id < 0 || id >= kNumTwo) {
    snprintf(buf, len, "invalid");
    return;
  }
  const TwoStepShape& t = kTwo[id];
  if (t.mr > 0)
    snprintf(buf, len, "2step:64x%d/%d+march%dxh%d+xcdband%s", t.ty, t.nt, t.mr, t.h, t.nts ? "+nts" : "");
  else
    snprintf(buf, len, "2step:64x%d/%d%s%s", t.ty, t.nt, t.map == 1 ? "+xcd8" : (t.map == 2 ? "+xcdband" : ""),
             t.nts ? "+nts" : "");
}

bool two_step_supported(const LatDesc& L) {
  return L.bc[E_LEFT] == BC_NSBC && L.bc[E_RIGHT] == BC_NSBC && L.bc[E_BOTTOM] == BC_NSBC &&
         L.bc[E_TOP] == BC_NSBC && L.nx >= 3 && L.ny >= 3;
}

template <int S, int TY, int NT, bool NTS, int MAP>
static hipError_t launch_two_t(const LatDesc& L, int parity, hipStream_t s) {
  const int tiles_x = (L.nx + TL_TX - 1) / TL_TX, tiles_y = (L.ny + TY - 1) / TY;
  dim3 grid(tiles_x, tiles_y);
  if (MAP == 1) grid = dim3(((tiles_x * tiles_y + 63) >> 6) * 64);
  if (MAP == 2) grid = dim3(((tiles_x * tiles_y + 7) >> 3) * 8);
  if (L.coll == COLL_MRT)
    k_two_step<S, TY, NT, NTS, COLL_MRT, MAP><<<grid, dim3(NT), 0, s>>>(L, parity, tiles_x, tiles_y);
  else
    k_two_step<S, TY, NT, NTS, COLL_BGK, MAP><<<grid, dim3(NT), 0, s>>>(L, parity, tiles_x, tiles_y);
  return hipGetLastError();
}

template <int S>
static hipError_t launch_two_s(const LatDesc& L, int parity, int id, hipStream_t s) {
  int k = 0;
#define X(a, b, c, d)                                               \
  if (id == k) return launch_two_t<S, a, b, c, d>(L, parity, s);   \
  ++k;
  LBM_TWO_STEP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_two_step(const LatDesc& L, int parity, int id, hipStream_t s) {
  // the two-step sweep has no closure path
  if (!two_step_supported(L) || (L.closure && L.net)) return hipErrorInvalidValue;
  if (id >= 0 && id < kNumTwo && kTwo[id].mr > 0) return launch_two_march(L, parity, id - (kNumTwo - kNumTwoMarch), s);
  switch (L.store) {
    case ST_F64: return launch_two_s<ST_F64>(L, parity, id, s);
    case ST_F32: return launch_two_s<ST_F32>(L, parity, id, s);
    case ST_F16: return launch_two_s<ST_F16>(L, parity, id, s);
    case ST_BF16: return launch_two_s<ST_BF16>(L, parity, id, s);
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ three-step kernel
// (shapes and kernel in lbm_threestep.h)
// the tile shapes first, then the marched ones (mr > 0: rows per round, h:
// chunk rows; non-temporal stores)
struct ThreeStepShape {
  int ty, nt;
  bool nts;
  int mr, h, pf;
};
static const ThreeStepShape kThree[] = {
#define X(a, b, c) {a, b, c, 0, 0, 0},
    LBM_THREE_STEP(X)
#undef X
#define X(a, m, b, h, p, n) {a, b, n, m, h, p},
    LBM_THREE_MARCH(X)
#undef X
};
static constexpr int kNumThree = sizeof(kThree) / sizeof(kThree[0]);
static constexpr int kNumMarch = 0
#define X(a, m, b, h, p, n) +1
    LBM_THREE_MARCH(X)
#undef X
    ;

bool three_step_is_march(int id) { return id >= 0 && id < kNumThree && kThree[id].mr > 0; }

int num_three_step() { return kNumThree; }

void three_step_name(int id, char* buf, size_t len) {
  if (id < 0 || id >= kNumThree) {
    snprintf(buf, len, "invalid");
    return;
  }
  // (the names are identifiers that callers keep: a march's is "+xcdband" from when its XCDs took bands)
  const ThreeStepShape& t = kThree[id];
  if (t.mr > 0)
    snprintf(buf, len, "3step:64x%d/%d+march%dxh%d%s+xcdband%s", t.ty, t.nt, t.mr, t.h, t.pf == 2 ? "+pf2" : "",
             t.nts ? "+nts" : "");
  else
    snprintf(buf, len, "3step:64x%d/%d+xcdband%s", t.ty, t.nt, t.nts ? "+nts" : "");
}

bool three_step_supported(const LatDesc& L, int id) {
  return id >= 0 && id < kNumThree && two_step_supported(L) && L.nx >= TL_TX && L.ny >= kThree[id].ty &&
         three_step_fits_store(L.store, id, L.closure && L.net);
}

// The first tile shape with a march shape's tile rows: it runs the march's edge
// tiles of a closure lattice, and the whole of a lattice too small for the march.
static int tile_shape_of(int id) {
  for (int k = 0; k < kNumThree; ++k)
    if (kThree[k].mr == 0 && kThree[k].ty == kThree[id].ty) return k;
  return -1;
}

// One launch of a tile or march shape, except on the learned closure, which
// takes its edge tiles with the network in a kernel of their own (both kernels read
// buffer `parity` and write disjoint parts of the other one).  With a second stream
// `side` that kernel runs there, forked from `s` after the work already on it
// (event `fork`) and joined back before what follows (event `join`); without one
// the kernels run in turn on `s`.
//
// The inner part splits in two: its border (the march items or inner tiles that
// share values with an edge tile) and its middle, which stays 3 nodes or more from
// every edge tile.  Launch n's edge tiles need launch n - 1's border and edge tiles,
// launch n's border needs launch n - 1's edge tiles, border and middle, and launch
// n's middle only what ran on s before it.  So s runs each launch's border first and
// records `fork` there: the edge tiles of the next launch run beside this launch's
// middle and need to end only before that launch's border is through (with kJoinDefer
// on every launch but the last and kJoinPrev on every launch but the first).  With the
// middle first, the edge tiles started after it and the next border waited for them.
// 2048^2 FP32 on the vortex, us per launch with the middle first and 64-wide edge tiles /
// as it is: most side nodes past the regime gate 117 / 96, few of them 93 / 92 (one
// fork and join per launch, border and middle in one kernel: 109 to 121 past the gate).
hipError_t launch_three_step(const LatDesc& L, int parity, int id, hipStream_t s, hipStream_t side, hipEvent_t fork,
                             hipEvent_t join, int flags) {
  if (!three_step_supported(L, id)) return hipErrorInvalidValue;
  if (kThree[id].mr > 0 && !march_fits(L, kThree[id].ty)) id = tile_shape_of(id);
  const bool closure = L.closure && L.net, march = kThree[id].mr > 0;
  const int mid = id - (kNumThree - kNumMarch);
  // part 0: all, 1: without the edge tiles, 3: the inner part's middle, 4: its border
  auto inner = [&](int part) {
    if (march) return launch_three_march(L, parity, mid, s, part == 0, part >= 3 ? part - 2 : 0);
    switch (L.store) {
      case ST_F64: return launch_three_s<ST_F64, false>(L, parity, id, s, part);
      case ST_F32: return launch_three_s<ST_F32, false>(L, parity, id, s, part);
      case ST_F16: return launch_three_s<ST_F16, false>(L, parity, id, s, part);
      case ST_BF16: return launch_three_s<ST_BF16, false>(L, parity, id, s, part);
    }
    return hipErrorInvalidValue;
  };
  auto edges = [&](hipStream_t es) {
    return march ? launch_march_ring_closure(L, parity, kThree[id].ty, es) : launch_three_step_closure(L, parity, id, es);
  };
  if (!closure) return inner(0);
  if (!(side && fork && join)) {
    const hipError_t e = edges(s);
    return e == hipSuccess ? inner(1) : e;
  }
  hipError_t e = hipSuccess;
  if (!(flags & kJoinPrev)) e = hipEventRecord(fork, s);
  if (e == hipSuccess) e = hipStreamWaitEvent(side, fork, 0);
  if (e == hipSuccess) e = edges(side);
  // s waits for the previous launch's edge tiles before join is recorded anew
  if ((flags & kJoinPrev) && e == hipSuccess) e = hipStreamWaitEvent(s, join, 0);
  if (e == hipSuccess) e = hipEventRecord(join, side);
  if (e == hipSuccess) e = inner(4);
  if ((flags & kJoinDefer) && e == hipSuccess) e = hipEventRecord(fork, s);
  if (e == hipSuccess) e = inner(3);
  if (!(flags & kJoinDefer) && e == hipSuccess) e = hipStreamWaitEvent(s, join, 0);
  return e;
}

// ------------------------------------------------------------------ ensemble
// Whether an ensemble's three-step sweep in tiles of `ty` rows marches its larger members (the rows
// that the single-lattice marches use), and in chunks of about how many rows.  256 members of 64^2 to 512^2
// in FP32, us per launch: tiles 505 to 520; marched in chunks of 18 / 29 / 40 / 62 / 96 rows 464 / 441 / 439 /
// 454 / 468 (12 rows, 768 threads) and 445 / 441 / 447 / 461 / 480 (8 rows).  Longer chunks recompute
// fewer rows, but leave the edge tiles of their own member to other times.
constexpr bool ens_marches(int ty) { return ty == 8 || ty == 12; }
constexpr int ens_march_rows(int ty) { return ty == 12 ? 40 : 29; }

// One block per entry of a device list of (member, tile) in block order (the
// host lays the list out so that each XCD takes short runs of neighbours).  The
// member's descriptor carries its collision model, read at run time.
template <int S, int TY, int NT, bool NTS>
__global__ __launch_bounds__(NT, two_step_waves<S>()) void k_ens_two_step(const LatDesc* __restrict__ descs,
                                                     const TwoTile* __restrict__ list, int parity) {
  const TwoTile t = list[blockIdx.x];
  const LatDesc L = descs[t.lat];
  two_step_tile<S, TY, NT, NTS, -1>(L, parity, t.txi, t.tyi);
}

int two_step_tile_rows(int id) { return id >= 0 && id < kNumTwo ? kTwo[id].ty : 0; }

int two_step_min_rows() {
  int m = kTwo[0].ty;
  for (int i = 1; i < kNumTwo; ++i) m = kTwo[i].ty < m ? kTwo[i].ty : m;
  return m;
}

// Three-step sweep over an ensemble's list (as k_ens_two_step).  An entry is a 64 x TY
// tile of a member (pad == 0); where the member is large enough to march
// (MarchGeom), its edge tiles (pad == -1, txi the number) and its strips' chunks (txi the
// strip, output rows tyi .. pad - 1) take the place of its tiles.
template <int S, int TY, int NT, bool NTS>
__global__ __launch_bounds__(NT, two_step_waves<S>()) void k_ens_three_step(const LatDesc* __restrict__ descs,
                                                       const TwoTile* __restrict__ list, int parity) {
  const TwoTile t = list[blockIdx.x];
  const LatDesc L = descs[t.lat];
  if constexpr (ens_marches(TY)) {
    if (t.pad > 0) {
      three_step_march<S, TY, TY - 1, NT, NTS, -1, 1, true>(L, parity, t.txi, t.tyi, t.pad);
      return;
    }
    int xo = t.txi * TL_TX, yo = t.tyi * TY, x0 = min(xo, L.nx - TL_TX), y0 = min(yo, L.ny - TY);
    if (t.pad < 0) {
      bool side;
      march_ring_pos<TY, TL_TX>(t.txi, L.nx, L.ny, MarchGeom(L.nx, L.ny, TY), x0, y0, xo, yo, side);
      if (side) {
        three_step_tile_at<S, EDGE_TX, 4 * TY, TY, NT, NTS, -1>(L, parity, x0, y0, xo, yo, 2);
        return;
      }
    }
    three_step_tile_at<S, TL_TX, TY, TY, NT, NTS, -1>(L, parity, x0, y0, xo, yo, 0);
  } else {
    three_step_tile<S, TY, NT, NTS, -1>(L, parity, t.txi, t.tyi);
  }
}

// The entries of member `lat` (nx x ny) in three-step shape `id`'s list, marched where `march` and its
// size allow.
void ens_three_step_items(int id, int lat, int nx, int ny, bool march, std::vector<TwoTile>& items) {
  const int ty = kThree[id].ty;
  const MarchGeom g(nx, ny, ty);
  if (march && ens_marches(ty) && g.ix > 0) {
    const int chunks = march_chunks(g.rows, ens_march_rows(ty));
    for (int b = 0; b < g.ring(); ++b) items.push_back({lat, b, 0, -1});
    for (int c = 0; c < chunks; ++c)
      for (int sx = 0; sx < g.ix; ++sx)
        items.push_back({lat, sx, ty + march_row(c, g.rows, chunks), ty + march_row(c + 1, g.rows, chunks)});
    return;
  }
  for (int j = 0; j < (ny + ty - 1) / ty; ++j)
    for (int i = 0; i < (nx + TL_TX - 1) / TL_TX; ++i) items.push_back({lat, i, j, 0});
}

int three_step_tile_rows(int id) { return id >= 0 && id < kNumThree ? kThree[id].ty : 0; }

int three_step_min_rows() {
  int m = kThree[0].ty;
  for (int i = 1; i < kNumThree; ++i) m = kThree[i].ty < m ? kThree[i].ty : m;
  return m;
}

template <int S>
static hipError_t launch_ens_three_s(int id, const LatDesc* d, const TwoTile* list, int n, int parity,
                                     hipStream_t s) {
  int k = 0;
#define X(a, b, c)                                                                        \
  if (id == k) {                                                                          \
    if constexpr (three_step_fits<S, a>()) {                                              \
      k_ens_three_step<S, a, b, c><<<dim3(n), dim3(b), 0, s>>>(d, list, parity);          \
      return hipGetLastError();                                                           \
    } else {                                                                              \
      return hipErrorInvalidValue;                                                        \
    }                                                                                     \
  }                                                                                       \
  ++k;
  LBM_THREE_STEP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_ens_three_step(int store, int id, const LatDesc* d, const TwoTile* list, int n, int parity,
                                 hipStream_t s) {
  if (n <= 0) return hipSuccess;
  switch (store) {
    case ST_F64: return launch_ens_three_s<ST_F64>(id, d, list, n, parity, s);
    case ST_F32: return launch_ens_three_s<ST_F32>(id, d, list, n, parity, s);
    case ST_F16: return launch_ens_three_s<ST_F16>(id, d, list, n, parity, s);
    case ST_BF16: return launch_ens_three_s<ST_BF16>(id, d, list, n, parity, s);
  }
  return hipErrorInvalidValue;
}

template <int S>
static hipError_t launch_ens_two_s(int id, const LatDesc* d, const TwoTile* list, int n, int parity,
                                   hipStream_t s) {
  int k = 0;
#define X(a, b, c, m)                                                                   \
  if (id == k) {                                                                        \
    k_ens_two_step<S, a, b, c><<<dim3(n), dim3(b), 0, s>>>(d, list, parity);            \
    return hipGetLastError();                                                           \
  }                                                                                     \
  ++k;
  LBM_TWO_STEP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_ens_two_step(int store, int id, const LatDesc* d, const TwoTile* list, int n, int parity,
                               hipStream_t s) {
  if (n <= 0) return hipSuccess;
  switch (store) {
    case ST_F64: return launch_ens_two_s<ST_F64>(id, d, list, n, parity, s);
    case ST_F32: return launch_ens_two_s<ST_F32>(id, d, list, n, parity, s);
    case ST_F16: return launch_ens_two_s<ST_F16>(id, d, list, n, parity, s);
    case ST_BF16: return launch_ens_two_s<ST_BF16>(id, d, list, n, parity, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm

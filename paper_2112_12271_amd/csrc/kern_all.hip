// kern_all.hip -- per-tile kernels of a batch launched once over the tiles
// of every dimension class: each tile's system selects the
// dimension-templated body (update, binning, placement, list build,
// forces).  One launch per kernel instead of one per class keeps the launch
// count of a batch iteration independent of how many dimensions it mixes.
#include "kernels.h"
#include "dispatch.h"

namespace hdmd {

#define HDMD_EACH_D(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)
// classes of the all-class list build and forces: the d = 9, 10 bodies need
// more registers than four waves per SIMD allow, so those classes keep
// launches of their own
#define HDMD_BUILD_D(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

// The rebuild chain's kernels (binning, placement, list build) run in
// every iteration but find work only in the systems that rebuild, often one
// of hundreds.  Their workgroups therefore test many tiles at once, one per
// lane (tile entry, system pointer, flags: three dependent loads), and then
// walk the tiles that rebuild; a workgroup's tiles are strided by the grid
// so that a rebuilding system's tiles spread over the workgroups.
__device__ inline bool tile_rebuilds(const Table* tab, const int2* tiles, int t, int n, int2& e,
                                     int dmax = kMaxD) {
  if (t >= n) return false;
  e = tiles[t];
  const SysDev* s = tab->sys[e.x];
  return running(s) && need_rebuild(s) && s->d <= dmax;
}

__global__ __launch_bounds__(kTile) void k_bin_all(KArgs a) {
  const int n = a.tab->n_atom[0], g = gridDim.x, lane = threadIdx.x;
  const int2* tiles = a.tab->atom_tiles[0];
  for (int base = blockIdx.x; base < n; base += 64 * g) {
    int2 e = make_int2(0, 0);
    unsigned long long m = __ballot(tile_rebuilds(a.tab, tiles, base + lane * g, n, e));
    while (m) {
      const int k = __builtin_ctzll(m);
      m &= m - 1;
      SysDev* s = uniform_ptr(a.tab->sys[__builtin_amdgcn_readlane(e.x, k)]);
      const int tile = __builtin_amdgcn_readlane(e.y, k);
      if (tile == 0 && lane == 0)
        atomicAdd(&a.tab->build_waves, s->wrap ? s->ntiles : s->ncells);
      switch (s->d) {
#define HDMD_CASE(DD)      \
  case DD:                 \
    bin_tile<DD>(s, tile); \
    break;
        HDMD_EACH_D(HDMD_CASE)
#undef HDMD_CASE
      }
    }
  }
}

__global__ __launch_bounds__(kTile) void k_fire_update_all(KArgs a) {
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile(a, t, s, tile)) break;
    if (!live(s) || s->mode != MODE_FIRE) continue;
    const bool mix = s->precision != 0, zero = s->c_zero != 0;
    const double dt = s->fdt, keep = s->c_keep, mx = s->c_mix;
    switch (s->d) {
#define HDMD_CASE(DD)                                                  \
  case DD:                                                             \
    if (mix) fire_update_tile<DD, true>(s, tile, dt, keep, mx, zero);  \
    else fire_update_tile<DD, false>(s, tile, dt, keep, mx, zero);     \
    break;
      HDMD_EACH_D(HDMD_CASE)
#undef HDMD_CASE
    }
  }
}

__global__ __launch_bounds__(kTile) void k_place_all(KArgs a) {
  const int n = a.tab->n_atom[0], g = gridDim.x, lane = threadIdx.x;
  const int2* tiles = a.tab->atom_tiles[0];
  for (int base = blockIdx.x; base < n; base += 64 * g) {
    int2 e = make_int2(0, 0);
    unsigned long long m = __ballot(tile_rebuilds(a.tab, tiles, base + lane * g, n, e));
    while (m) {
      const int k = __builtin_ctzll(m);
      m &= m - 1;
      SysDev* s = uniform_ptr(a.tab->sys[__builtin_amdgcn_readlane(e.x, k)]);
      const int tile = __builtin_amdgcn_readlane(e.y, k);
      const bool mix = s->precision != 0;
      switch (s->d) {
#define HDMD_CASE(DD)                          \
  case DD:                                     \
    if (mix) place_tile<DD, float>(s, tile);   \
    else place_tile<DD, double>(s, tile);      \
    break;
        HDMD_EACH_D(HDMD_CASE)
#undef HDMD_CASE
      }
    }
  }
}

// FIRE forces of every class d <= kBuildAllMaxD (larger d: per-class launches)
template <bool MORSE>
__global__ __launch_bounds__(kTile) void k_force_all(KArgs a, int fire) {
  __shared__ double sh[kPart];
  __shared__ vd2 stage[kStage16];
  for (int t = xcd_tile(blockIdx.x, gridDim.x);; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile(a, t, s, tile)) break;
    if (!live(s) || (s->potential == kPotMorse) != MORSE || s->lpa != 1) continue;
    if (fire && s->mode != MODE_FIRE) continue;
    const bool mix = s->precision != 0;
    switch (s->d) {
#define HDMD_CASE(DD)                                           \
  case DD:                                                      \
    if (mix) force_tile<DD, true, 1, MORSE>(s, tile, fire, sh, stage); \
    else force_tile<DD, false, 1, MORSE>(s, tile, fire, sh, stage);    \
    break;
      HDMD_BUILD_D(HDMD_CASE)
#undef HDMD_CASE
    }
  }
}

// Verlet-list build of every rebuilding system with d <= kBuildAllMaxD (the
// d = 9, 10 bodies need more registers than four waves per SIMD allow, so
// those classes keep launches of their own): a subcell is one wave's work
// (four such per workgroup), and so is an atom tile of a system of the circle
// form.  One launch per stencil radius present (RAD 1: subcells of side >=
// r_l,max; RAD 2: half-size subcells), each passing over the subcells of the
// other radius.
//
// Few systems of a batch rebuild in one iteration, and a small one has fewer
// tiles than the card has SIMDs: the launch then lasts as long as one wave's
// chain of dependent loads.  When the rebuilding systems come to at most
// kSplitWaves waves, a wave takes a quarter of a tile's home atoms (the rows
// are the same).  Batch of 24 minimisations: 60.4 -> 53.7 ms.  Sharing a
// subcell's home atoms in the same way costs three times its work: the rows'
// set-up is repeated (60.5 ms).
constexpr int kSplitWaves = 2048;

template <int RAD>
__global__ __launch_bounds__(256, 4) void k_build_all(KArgs a) {
  __shared__ BuildLds<RAD> lds[4];
  static_assert(sizeof(WrapLds) <= sizeof(BuildLds<RAD>), "one LDS area serves both builds");
  cTable* tab = (cTable*)a.tab;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nnw = tab->n_cell[0];
  cint2* tiles = (cint2*)tab->cell_tiles[0];
  // this wave's tiles are strided by the waves of the launch
  const int g = gridDim.x * 4, me = xcd_tile(blockIdx.x, gridDim.x) * 4 + wv;
  for (int base = me; base < nnw; base += 64 * g) {
    int2 e;
    unsigned long long mk = __ballot(
        tile_rebuilds(a.tab, a.tab->cell_tiles[0], base + lane * g, nnw, e, kBuildAllMaxD));
    while (mk) {
      const int idx = base + __builtin_ctzll(mk) * g;
      mk &= mk - 1;
      SysDev* s = tab->sys[tiles[idx].x];
      cSys* c = (cSys*)s;
      const int hc = tiles[idx].y;
      if (c->reach != RAD) continue;
      const int mode = c->bmode;
      switch (c->d) {
#define HDMD_CASE(DD)                                                                              \
  case DD:                                                                                         \
    if (RAD == 1 && mode == BUILD_SPARSE)                                                          \
      build_mf_tile<DD, RAD, RAD == 1 ? BUILD_SPARSE : BUILD_DENSE>(s, hc, 0, 1, &lds[wv]); \
    else build_mf_tile<DD, RAD, BUILD_DENSE>(s, hc, 0, 1, &lds[wv]);                      \
    break;
        HDMD_BUILD_D(HDMD_CASE)
#undef HDMD_CASE
      }
    }
  }
  if constexpr (RAD == 1) {
    const int sh = tab->build_waves <= kSplitWaves ? 2 : 0;  // log2 of the waves per tile
    const int nat = tab->n_atom[0] << sh;
    cint2* at = (cint2*)tab->atom_tiles[0];
    for (int base = me; base < nat; base += 64 * g) {
      int2 e = make_int2(0, 0);
      bool act = tile_rebuilds(a.tab, a.tab->atom_tiles[0], (base + lane * g) >> sh, nat >> sh, e,
                               kBuildAllMaxD);
      if (act) act = a.tab->sys[e.x]->wrap != 0;
      unsigned long long mk = __ballot(act);
      while (mk) {
        const int idx = base + __builtin_ctzll(mk) * g;
        mk &= mk - 1;
        SysDev* s = tab->sys[at[idx >> sh].x];
        const int hb = at[idx >> sh].y * 64 + (idx & ((1 << sh) - 1)) * 16;
        switch (((cSys*)s)->d) {
#define HDMD_CASE(DD)                                                                  \
  case DD:                                                                             \
    if (sh) build_wrap_tile<DD, 1>(s, hb, 16, reinterpret_cast<WrapLds*>(&lds[wv]));       \
    else build_wrap_tile<DD, 4>(s, hb, kTile, reinterpret_cast<WrapLds*>(&lds[wv]));          \
    break;
          HDMD_BUILD_D(HDMD_CASE)
#undef HDMD_CASE
        }
      }
    }
  }
}

void launch_build_all(const KArgs& a, int grid, int reach, hipStream_t st) {
  if (reach == 2) k_build_all<2><<<grid, 256, 0, st>>>(a);
  else k_build_all<1><<<grid, 256, 0, st>>>(a);
}
void launch_bin_all(const KArgs& a, int grid, hipStream_t st) { k_bin_all<<<grid, kTile, 0, st>>>(a); }
void launch_force_all(const KArgs& a, int grid, int fire, bool morse, hipStream_t st) {
  if (morse) k_force_all<true><<<grid, kTile, 0, st>>>(a, fire);
  else k_force_all<false><<<grid, kTile, 0, st>>>(a, fire);
}
void launch_fire_update_all(const KArgs& a, int grid, hipStream_t st) {
  k_fire_update_all<<<grid, kTile, 0, st>>>(a);
}
void launch_place_all(const KArgs& a, int grid, hipStream_t st) {
  k_place_all<<<grid, kTile, 0, st>>>(a);
}

}  // namespace hdmd

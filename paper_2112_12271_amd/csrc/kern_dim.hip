// kern_dim.hip -- instantiates the kernels for one dimension HDMD_DIM and
// exports their launchers.  Built once per d = 2..10.
#include "kernels.h"
#include "dispatch.h"

#ifndef HDMD_DIM
#error "HDMD_DIM must be defined"
#endif

namespace hdmd {
namespace {
constexpr int D = HDMD_DIM;

void l_load(bool mix, SysDev* s, int grid, hipStream_t st, const double* pos, const double* diam,
            const double* vel) {
  if (mix) k_load<D, float><<<grid, kTile, 0, st>>>(s, pos, diam, vel);
  else k_load<D, double><<<grid, kTile, 0, st>>>(s, pos, diam, vel);
}
void l_unload(bool mix, const SysDev* s, int grid, hipStream_t st, double* pos, double* vel,
              double* force) {
  if (mix) k_unload<D, float><<<grid, kTile, 0, st>>>(s, pos, vel, force);
  else k_unload<D, double><<<grid, kTile, 0, st>>>(s, pos, vel, force);
}
void l_same_state(bool mix, SysDev* s, int grid, hipStream_t st, const double* pos, const double* vel,
                  const double* diam) {
  if (mix) k_same_state<D, float><<<grid, kTile, 0, st>>>(s, pos, vel, diam);
  else k_same_state<D, double><<<grid, kTile, 0, st>>>(s, pos, vel, diam);
}
void l_disp_restart(SysDev* s, int grid, hipStream_t st) {
  k_disp_restart<D><<<grid, kTile, 0, st>>>(s);
}
void l_bin(const KArgs& a, int grid, hipStream_t st) { k_bin<D><<<grid, kBinBlock, 0, st>>>(a); }
void l_place(bool mix, const KArgs& a, int grid, hipStream_t st) {
  if (mix) k_place<D, float><<<grid, 256, 0, st>>>(a);
  else k_place<D, double><<<grid, 256, 0, st>>>(a);
}
void l_build(int reach, int mode, int G, const KArgs& a, int grid, hipStream_t st) {
  if (reach == 2) {
    // half-size subcells, 5^d stencil
    if (G <= 1) k_build_mf<D, 1, 2, BUILD_DENSE><<<grid, 64, 0, st>>>(a);
    else if (G == 2) k_build_mf<D, 2, 2, BUILD_DENSE><<<grid, 128, 0, st>>>(a);
    else k_build_mf<D, 4, 2, BUILD_DENSE><<<grid, 256, 0, st>>>(a);
  } else if (mode == BUILD_DENSE) {
    if (G <= 1) k_build_mf<D, 1, 1, BUILD_DENSE><<<grid, 64, 0, st>>>(a);
    else if (G == 2) k_build_mf<D, 2, 1, BUILD_DENSE><<<grid, 128, 0, st>>>(a);
    else k_build_mf<D, 4, 1, BUILD_DENSE><<<grid, 256, 0, st>>>(a);
  } else {
    if (G <= 1) k_build_mf<D, 1, 1, BUILD_SPARSE><<<grid, 64, 0, st>>>(a);
    else if (G == 2) k_build_mf<D, 2, 1, BUILD_SPARSE><<<grid, 128, 0, st>>>(a);
    else k_build_mf<D, 4, 1, BUILD_SPARSE><<<grid, 256, 0, st>>>(a);
  }
}
void l_build_wrap(int homes, const KArgs& a, int grid, hipStream_t st) {
  if (homes <= 16) k_build_wrap<D, 1><<<grid, 64, 0, st>>>(a, homes);
  else k_build_wrap<D, 4><<<grid, 64, 0, st>>>(a, homes);
}
template <bool MIX, int LPA, bool MORSE = false>
void force_lpa(const KArgs& a, int grid, int fire, hipStream_t st) {
  k_force<D, MIX, LPA, MORSE><<<grid, kTile * LPA, 0, st>>>(a, fire);
}
template <bool MIX, int LPA, bool MORSE = false>
void step_lpa(const KArgs& a, int grid, hipStream_t st) {
  k_step<D, MIX, LPA, MORSE><<<grid, kTile * LPA, 0, st>>>(a);
}
// Morse systems run one lane per atom
void l_force(bool mix, int lpa, bool morse, const KArgs& a, int grid, int fire, hipStream_t st) {
  if (morse) {
    if (mix) force_lpa<true, 1, true>(a, grid, fire, st);
    else force_lpa<false, 1, true>(a, grid, fire, st);
  } else if (mix) {
    if (lpa >= 4) force_lpa<true, 4>(a, grid, fire, st);
    else if (lpa == 2) force_lpa<true, 2>(a, grid, fire, st);
    else force_lpa<true, 1>(a, grid, fire, st);
  } else {
    if (lpa >= 4) force_lpa<false, 4>(a, grid, fire, st);
    else if (lpa == 2) force_lpa<false, 2>(a, grid, fire, st);
    else force_lpa<false, 1>(a, grid, fire, st);
  }
}
void l_step(bool mix, int lpa, bool morse, const KArgs& a, int grid, hipStream_t st) {
  if (morse) {
    if (mix) step_lpa<true, 1, true>(a, grid, st);
    else step_lpa<false, 1, true>(a, grid, st);
  } else if (mix) {
    if (lpa >= 4) step_lpa<true, 4>(a, grid, st);
    else if (lpa == 2) step_lpa<true, 2>(a, grid, st);
    else step_lpa<true, 1>(a, grid, st);
  } else {
    if (lpa >= 4) step_lpa<false, 4>(a, grid, st);
    else if (lpa == 2) step_lpa<false, 2>(a, grid, st);
    else step_lpa<false, 1>(a, grid, st);
  }
}
void l_fire_update(bool mix, const KArgs& a, int grid, hipStream_t st) {
  if (mix) k_fire_update<D, true><<<grid, kTile, 0, st>>>(a);
  else k_fire_update<D, false><<<grid, kTile, 0, st>>>(a);
}
void l_vanhove(const SysDev* s, int grid, hipStream_t st, int nbins, double w,
               unsigned long long* hist, double* disp) {
  k_vanhove<D><<<grid, kTile, 0, st>>>(s, nbins, w, hist, disp);
}
void l_swap_de(const SysDev* s, hipStream_t st, const long long* ctl, const int32_t* off_in,
               int64_t n_att, const int32_t* pairs, const int32_t* slot_of, double* de,
               unsigned long long* conf) {
  k_swap_de<D><<<kSwapBatch, 1024, 0, st>>>(s, ctl, off_in, n_att, pairs, slot_of, de, conf);
}
void l_swap_settle(SysDev* s, hipStream_t st, long long* ctl, const int32_t* off_in,
                   int32_t* off_out, int64_t n_att, const int32_t* pairs, const double* u, double T,
                   const int32_t* slot_of, const double* de, const unsigned long long* conf,
                   int32_t* acc, double* diam) {
  k_swap_settle<D><<<1, kSwapBatch, 0, st>>>(s, ctl, off_in, off_out, n_att, pairs, u, T, slot_of, de,
                                       conf, acc, diam);
}
const DKernels table = {l_load, l_unload, l_same_state, l_disp_restart, l_bin, l_place, l_build, l_build_wrap, l_force, l_step,
                        l_fire_update, l_vanhove, l_swap_de, l_swap_settle};
}  // namespace

#define HDMD_CAT2(a, b) a##b
#define HDMD_CAT(a, b) HDMD_CAT2(a, b)
const DKernels* HDMD_CAT(dkernels_d, HDMD_DIM)() { return &table; }

}  // namespace hdmd

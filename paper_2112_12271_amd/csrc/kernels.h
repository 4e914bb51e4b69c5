// kernels.h -- the gfx950 kernels of the hot path, templated on the dimension D.
//
//  k_load        caller [n][d] arrays -> internal buffers (wrap, validate)
//  k_bin         subcell of every atom + occupancy counts      (Sec. II.C)
//  k_scatter     counting-sort placement by subcell            (common.hip)
//  k_place       order within the subcell, permutation of every per-atom
//                array, reference positions, list-build records; finalisation
//  k_build_mf, k_build_wrap  Verlet rows over the linked subcells (Sec. II.C, Fig. 1)
//  k_force       pair forces and energy (+ FIRE reductions)    (Sec. II.B)
//  k_step        fused velocity-Verlet step + rebuild trigger (Sec. II.B/II.C)
//  k_fire_update semi-implicit Euler FIRE update
//  k_unload      internal -> caller order
//  k_vanhove     unwrapped displacements and the self van Hove histogram
//  k_swap_de, k_swap_settle  SWAP Monte Carlo in batches (Sec. II.D)
#pragma once
#include <type_traits>

#include "hdmd_dev.h"

namespace hdmd {

// ---------------------------------------------------------------------------
// load / unload
// ---------------------------------------------------------------------------
template <int D, typename VT>
__global__ __launch_bounds__(kTile) void k_load(SysDev* s, const double* __restrict__ pos,
                                                const double* __restrict__ diam,
                                                const double* __restrict__ vel) {
  int i = blockIdx.x * kTile + threadIdx.x;
  if (i >= s->npad) return;
  const int cur = s->xcur, pc = s->pcur, npad = s->npad;
  double* xo = s->x[cur ^ 1];
  VT* vo = reinterpret_cast<VT*>(s->v[pc]);
  double x[D];
  if (i >= s->n) {
#pragma unroll
    for (int k = 0; k < D; k++) {
      x[k] = 0.0;
      vo[(size_t)k * npad + i] = VT(0);
    }
    store_rec<D>(xo, i, x, 0.0);
    s->oid[pc][i] = -1;
    return;
  }
  const double L = s->L, h = s->hL;
  int err = 0;
#pragma unroll
  for (int k = 0; k < D; k++) {
    double t = pos[(size_t)i * D + k];
    if (!isfinite(t)) {
      err |= ERR_NONFINITE;
      t = 0.0;
    } else if (t < -3.0 * h || t >= 3.0 * h) {
      err |= ERR_ARG;
      t = 0.0;
    }
    x[k] = wrap1(t, L, h);
    double u = vel ? vel[(size_t)i * D + k] : 0.0;
    if (!isfinite(u)) {
      err |= ERR_NONFINITE;
      u = 0.0;
    }
    vo[(size_t)k * npad + i] = VT(u);
  }
  double sg = diam[i];
  if (!isfinite(sg)) {
    err |= ERR_NONFINITE;
    sg = 0.0;
  } else if (!(sg > 0.0) || sg > s->sigma_max) {
    err |= ERR_ARG;
  }
  store_rec<D>(xo, i, x, sg);
  s->oid[pc][i] = i;
  if (err) atomicOr(&s->err, err);
}

template <int D, typename VT>
__global__ __launch_bounds__(kTile) void k_unload(const SysDev* s, double* __restrict__ pos,
                                                  double* __restrict__ vel,
                                                  double* __restrict__ force) {
  int p = blockIdx.x * kTile + threadIdx.x;
  if (p >= s->n) return;
  const int cur = s->xcur, pc = s->pcur, npad = s->npad;
  int a = s->oid[pc][p];
  if (pos) {
    double x[D];
    load_x<D>(s->x[cur], p, x);
#pragma unroll
    for (int k = 0; k < D; k++) pos[(size_t)a * D + k] = x[k];
  }
  if (vel) {
    const VT* v = reinterpret_cast<const VT*>(s->v[pc]);
#pragma unroll
    for (int k = 0; k < D; k++) vel[(size_t)a * D + k] = double(v[(size_t)k * npad + p]);
  }
  if (force) {
    const VT* f = reinterpret_cast<const VT*>(s->f);
#pragma unroll
    for (int k = 0; k < D; k++) force[(size_t)a * D + k] = double(f[(size_t)k * npad + p]);
  }
}

// Whether the caller's arrays (positions, velocities, diameters in caller
// order) are bit for bit the state the workspace holds, as the last unload
// wrote them; any difference sets s->differ.
template <int D, typename VT>
__global__ __launch_bounds__(kTile) void k_same_state(SysDev* s, const double* __restrict__ pos,
                                                      const double* __restrict__ vel,
                                                      const double* __restrict__ diam) {
  const int p = blockIdx.x * kTile + threadIdx.x;
  if (p >= s->n) return;
  const int pc = s->pcur, npad = s->npad;
  const int a = s->oid[pc][p];
  double x[D], sg;
  load_rec<D>(s->x[s->xcur], p, x, sg);
  const VT* v = reinterpret_cast<const VT*>(s->v[pc]);
  bool same = diam[a] == sg;
#pragma unroll
  for (int k = 0; k < D; k++) {
    same = same && pos[(size_t)a * D + k] == x[k];
    same = same && vel[(size_t)a * D + k] == double(v[(size_t)k * npad + p]);
  }
  if (!same) atomicOr(&s->differ, 1);
}

// The displacement observables of a continued run start from zero: the
// displacement up to the last build is set to minus the part since it.
template <int D>
__global__ __launch_bounds__(kTile) void k_disp_restart(SysDev* s) {
  const int p = blockIdx.x * kTile + threadIdx.x;
  if (p >= s->npad) return;
  const int pc = s->pcur, npad = s->npad;
  double x[D];
  load_x<D>(s->x[s->xcur], p, x);
#pragma unroll
  for (int k = 0; k < D; k++) {
    const size_t o = (size_t)k * npad + p;
    s->disp[pc][o] = p < s->n ? -min_image(x[k] - s->xref[o], s->L, s->hL) : 0.0;
  }
}

// Unwrapped displacement of every atom since the MD call's step 0 (the
// displacement up to the last build plus the minimum image of x - x_ref),
// written in caller order to disp ([n][d], optional), and the histogram of
// |dr| behind the self part of the van Hove function (eq. VGC, Sec. II.E):
// hist[b] counts b w <= |dr| < (b+1) w, hist[nbins] the atoms beyond.
template <int D>
__global__ __launch_bounds__(kTile) void k_vanhove(const SysDev* s, int nbins, double w,
                                                   unsigned long long* __restrict__ hist,
                                                   double* __restrict__ disp) {
  const int p = blockIdx.x * kTile + threadIdx.x;
  if (p >= s->n) return;
  const int pc = s->pcur, npad = s->npad;
  const double L = s->L, h = s->hL;
  double x[D];
  load_x<D>(s->x[s->xcur], p, x);
  const int a = s->oid[pc][p];
  double r2 = 0.0;
#pragma unroll
  for (int k = 0; k < D; k++) {
    const size_t o = (size_t)k * npad + p;
    const double dk = s->disp[pc][o] + min_image(x[k] - s->xref[o], L, h);
    if (disp) disp[(size_t)a * D + k] = dk;
    r2 = __builtin_fma(dk, dk, r2);
  }
  if (hist) {
    const double q = floor(sqrt(r2) / w);
    const int b = q < (double)nbins ? (int)q : nbins;
    atomicAdd(hist + b, 1ull);
  }
}

// ---------------------------------------------------------------------------
// subcell binning: C_k = floor((x_k + L/2) n/L) clamped, I = sum C_k n^(d-1-k)
// ---------------------------------------------------------------------------
template <int D>
__device__ inline int flat_cell(const SysDev* s, const double (&x)[D]) {
  const int nc = s->ncell;
  const double h = s->hL, inv = s->inv_lsc;
  int I = 0;
#pragma unroll
  for (int k = 0; k < D; k++) {
    int c = (int)floor((x[k] + h) * inv);
    c = c < 0 ? 0 : (c > nc - 1 ? nc - 1 : c);
    I = I * nc + c;
  }
  return I;
}

// Loads and stores that pass by the caches that are not coherent over the
// device: values handed from workgroup to workgroup of one launch.
__device__ inline int load_agent(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_agent(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One atom tile (a wave) of a system that rebuilds: subcell index and arrival
// rank.  The wave adds to a subcell's count once for all its atoms there: in
// the order of the last build most of a wave's atoms share a few subcells, and
// one addition each made the counts the bottleneck (d = 8, N = 131072, 256
// subcells: 300 us of same-address additions).  It gathers the subcells of
// kBinGather lanes that way; the atoms left over, of waves whose atoms are
// scattered over many subcells (a first build in the caller's order, few atoms
// per subcell), are added one by one: gathering all 64 took 7 us of a first
// build of N = 1152 (k_bin 10.6 us; 3.2 without).  Eight were too few for runs
// (d = 4, N = 65536, 6.6 atoms per subcell: 12.99 ms, 12.94 with sixteen).
constexpr int kBinGather = 16;
template <int D>
__device__ inline void bin_tile(SysDev* s, int tile) {
  const int lane = threadIdx.x & 63;
  if (tile == 0 && lane == 0) {
    s->rx = s->xcur;
    s->rp = s->pcur;
  }
  const int i = tile * kTile + lane;
  const bool vi = i < s->n;
  int c = -1;
  if (vi) {
    double x[D];
    load_x<D>(s->x[s->xcur ^ 1], i, x);
    if (s->mode == MODE_MD) {
      // fold the displacement since the last build into the unwrapped
      // displacement (it stays below L/2 between builds, so the minimum image
      // is the true one)
      double* dp = s->disp[s->pcur];
      const size_t np = s->npad;
#pragma unroll
      for (int k = 0; k < D; k++)
        dp[k * np + i] += min_image(x[k] - s->xref[k * np + i], s->L, s->hL);
    }
    c = flat_cell<D>(s, x);
  }
  int rk = 0, lead = lane, cnt = 1;
  unsigned long long todo = __ballot(vi);
  for (int g = 0; g < kBinGather && todo; g++) {
    const int l = __builtin_ctzll(todo);
    const unsigned long long m = __ballot(c == __builtin_amdgcn_readlane(c, l));
    if (m >> lane & 1) {
      rk = __popcll(m & ((1ull << lane) - 1));
      lead = l;
      cnt = __popcll(m);
    }
    todo &= ~m;
  }
  int base = 0;
  if (vi && rk == 0) base = atomicAdd(&s->cell_count[c], cnt);
  base = __shfl(base, lead);
  if (vi) {
    store_agent(s->cell_of + i, c);
    store_agent(s->rank + i, base + rk);
  }
}

// Counting-sort placement of atom i, arrival rank r in subcell c: slot =
// start(subcell) + rank.  key: the atom's place in its subcell's order.
__device__ inline void scatter_atom(SysDev* s, int i, int c, int r) {
  const int slot = cell_start(s, c) + r;
  int key = s->oid[s->pcur][i];
  if (s->ysort) {
    // the offset along the last axis exactly as k_place quantises it (caller
    // ids below 2^23)
    const double xl = s->x[s->xcur ^ 1][(size_t)i * rec_stride(s->d) + s->d - 1];
    key |= (quant8(xl - last_centre(s, c), s->qinv) + 128) << 23;
  }
  s->key[slot] = key;
  s->src[slot] = i;
}

// Exclusive prefix of the subcell occupancies by one workgroup of kBinBlock
// threads, 1024 subcells per wave and pass (sixteen independent wave scans).
// sh: kBinBlock / 64 words.
__device__ inline void scan_cells(SysDev* s, int* sh) {
  constexpr int W = kBinBlock / 64, PER = 16;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nc = s->ncells;
  int carry = 0;
  for (int b = 0; b < nc; b += kBinBlock * PER) {
    const int c0 = b + w * 64 * PER + lane;
    int v[PER], x[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) v[u] = c0 + 64 * u < nc ? load_agent(s->cell_count + c0 + 64 * u) : 0;
#pragma unroll
    for (int u = 0; u < PER; u++) x[u] = v[u];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
      for (int u = 0; u < PER; u++) {
        const int y = __shfl_up(x[u], o);
        if (lane >= o) x[u] += y;
      }
    }
    int tot = 0;
#pragma unroll
    for (int u = 0; u < PER; u++) {
      const int t = __builtin_amdgcn_readlane(x[u], 63);
      x[u] += tot - v[u];
      tot += t;
    }
    if (lane == 0) sh[w] = tot;
    __syncthreads();
    int all = 0;
    for (int q = 0; q < W; q++) {
      const int t = sh[q];
      if (q < w) carry += t;
      else all += t;
    }
#pragma unroll
    for (int u = 0; u < PER; u++)
      if (c0 + 64 * u < nc) s->cell_local[c0 + 64 * u] = carry + x[u];
    carry += all;
    __syncthreads();
  }
  for (int ch = tid; ch < s->nchunks; ch += kBinBlock) s->chunk_off[ch] = 0;
  if (tid == 0) s->max_row = 0;
}

// The binning of a system alone, and in its last workgroup to end (by
// ticket) the prefix sums of the counts, and for few atoms the scatter too
// (bin_scans, bin_scatters).
template <int D>
__global__ __launch_bounds__(kBinBlock) void k_bin(KArgs a) {
  __shared__ int sh[kBinBlock / 64];
  SysDev* s = a.single;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool rb = running(s) && need_rebuild(s);
  if (blockIdx.x == 0 && tid == 0) s->rb = rb;
  if (!rb) return;
  const int nt = s->ntiles, n = s->n;
  for (int t = blockIdx.x * (kBinBlock / 64) + w; t < nt; t += gridDim.x * (kBinBlock / 64))
    bin_tile<D>(s, t);
  if (!bin_scans(a.fin, n, s->nchunks)) return;
  // every value the last workgroup reads of the others' went out past the
  // caches (additions, store_agent); it has arrived when the wave's count of
  // outstanding accesses is zero, so that no cache is written back here
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) sh[0] = atomicAdd(&s->ticket, 1) == (int)gridDim.x - 1;
  __syncthreads();
  if (!sh[0]) return;
  __syncthreads();
  if (tid == 0) s->ticket = 0;
  scan_cells(s, sh);
  if (!bin_scatters(a.fin, n, s->nchunks)) return;
  __threadfence_block();
  __syncthreads();
  for (int b = tid; b < n; b += 4 * kBinBlock) {
    int c[4], r[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int i = min(b + u * kBinBlock, n - 1);
      c[u] = load_agent(s->cell_of + i);
      r[u] = load_agent(s->rank + i);
    }
#pragma unroll
    for (int u = 0; u < 4; u++)
      if (b + u * kBinBlock < n) scatter_atom(s, b + u * kBinBlock, c[u], r[u]);
  }
}

// ---------------------------------------------------------------------------
// subcell order and permutation of the atom arrays
// ---------------------------------------------------------------------------
typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
__device__ inline unsigned h2u(hv2 v) { return __builtin_bit_cast(unsigned, v); }
__device__ inline hv2 u2h(unsigned v) { return __builtin_bit_cast(hv2, v); }

// The candidate slots of an atom (see the list build below) from its int8 offsets and C.
template <int D>
__device__ inline void cand_record(const int (&q)[D], int C, unsigned (&w)[8]) {
  _Float16 sl[16];
#pragma unroll
  for (int k = 0; k < 16; k++) sl[k] = (_Float16)0;
  sl[0] = (_Float16)(short)(2 * q[D - 1]);
  sl[1] = (_Float16)2048;
  sl[2] = sl[3] = (_Float16)1;
#pragma unroll
  for (int k = 0; k < D - 1; k++) sl[4 + k] = (_Float16)(short)(2 * q[k]);
  sl[D + 3] = (_Float16)(short)(C >> 11);
  sl[D + 4] = (_Float16)(short)(C & 2047);
#pragma unroll
  for (int t = 0; t < 8; t++) w[t] = h2u(hv2{sl[2 * t], sl[2 * t + 1]});
}

typedef _Float16 hv8 __attribute__((ext_vector_type(8)));
template <int D>
struct WrapRec {
  static constexpr int SLOTS = 2 * D + 2 <= 16 ? 16 : 24;
  static constexpr int WORDS = SLOTS / 2;            // record words
  static constexpr int LW = SLOTS == 16 ? 2 : 4;     // words per lane and operand
};

// f16 rounding: every cos and sin is off by at most 2^-12 + 2^-24, so the sum
// of 2 d products by less than 2 d * 2 * 2^-12 * (|cos| + |sin|)/2 <= 1.42 d
// 2^-11, and each share by 2^-11 d (|t| < 2 d); the margin of a share covers
// half of the first and its own, doubled.
__host__ __device__ constexpr double wrap_margin(int d) { return d * (1.42 / 2048.0 + 2.0 / 2048.0); }

template <int D>
__device__ inline void wrap_record(const SysDev* s, const double (&x)[D], double sg, int32_t* out) {
  typedef WrapRec<D> R;
  _Float16 sl[R::SLOTS];
#pragma unroll
  for (int k = 0; k < R::SLOTS; k++) sl[k] = (_Float16)0;
  const double two_pi = 6.283185307179586;
#pragma unroll
  for (int k = 0; k < D; k++) {
    const float th = (float)(x[k] / s->L * two_pi);
    sl[2 * k] = (_Float16)cosf(th);
    sl[2 * k + 1] = (_Float16)sinf(th);
  }
  const double a = two_pi / s->L * 0.5 * (s->cutoff * sg + s->skin);
  sl[2 * D] = (_Float16)1;
  // a share below the f16 range passes every pair, as -2 d does
  sl[2 * D + 1] = (_Float16)(float)fmax(0.5 * D - a * a - wrap_margin(D), -2.0 * D);
#pragma unroll
  for (int t = 0; t < R::WORDS; t++) out[t] = (int)h2u(hv2{sl[2 * t], sl[2 * t + 1]});
}

// One atom tile (a wave) of the placed slots: an atom's place in its subcell
// is the number of smaller keys there (caller id, or, with ysort, the
// quantised offset along the last axis and then caller id; all distinct), and
// every per-atom array is permuted into that order.  Counting reads the few
// keys of a subcell once per atom, from the caches; a bitonic sort per
// subcell, one workgroup for each, was a chain of barriers over mostly idle
// lanes (d = 4, N = 65536, 6.6 atoms per subcell: 80 us).
template <int D, typename VT>
__device__ inline void place_tile(SysDev* s, int tile) {
  constexpr bool MIX = sizeof(VT) == 4;
  const int lane = threadIdx.x & 63, nc = s->ncell, ncells = s->ncells, n = s->n;
  for (int c = tile * kTile + lane; c < ncells; c += s->ntiles * kTile) {
    s->cell_count[c] = 0;  // ready for the next build
    s->cell_flat[c] = cell_start(s, c);
  }
  if (tile == 0 && lane == 0) s->cell_flat[ncells] = n;
  const int p = tile * kTile + lane;
  if (p >= n) return;
  const int key = s->key[p], src = s->src[p];
  const int c = s->cell_of[src];
  const int cur = s->rx, pc = s->rp, pn = pc ^ 1, npad = s->npad;
  double x[D], sg;
  load_rec<D>(s->x[cur ^ 1], src, x, sg);
  const int s0 = cell_start(s, c), cnt = cell_start(s, c + 1) - s0;
  const HDMD_GLOBAL int* kc = gbl(s->key) + s0;
  int dst = s0;
  for (int k = 0; k < cnt; k += 8) {
    int o[8];
#pragma unroll
    for (int u = 0; u < 8; u++) o[u] = kc[min(k + u, cnt - 1)];
#pragma unroll
    for (int u = 0; u < 8; u++) dst += (k + u < cnt) & (o[u] < key);
  }
  const VT* vin = reinterpret_cast<const VT*>(s->v[pc]);
  VT* vout = reinterpret_cast<VT*>(s->v[pn]);
  const bool md = s->mode == MODE_MD;
  const double* din = s->disp[pc];
  double* dout = s->disp[pn];
  store_rec<D>(s->x[cur], dst, x, sg);
  if (MIX) store_q<D>(s->q[cur], dst, x, sg, s->hL, s->fxscale);
#pragma unroll
  for (int k = 0; k < D; k++) {
    s->xref[(size_t)k * npad + dst] = x[k];
    vout[(size_t)k * npad + dst] = vin[(size_t)k * npad + src];
    if (md) dout[(size_t)k * npad + dst] = din[(size_t)k * npad + src];
  }
  if (s->wrap) {
    // slots on the circle (the circle form of the list build)
    wrap_record<D>(s, x, sg, s->qc16 + (size_t)dst * WrapRec<D>::WORDS);
  } else {
    // the candidate slots of the matrix-core build, from the offsets to the
    // subcell's centre
    int qv[D], Q = 0, u = c;
#pragma unroll
    for (int k = D - 1; k >= 0; k--) {
      const double cen = k == D - 1 ? last_centre(s, c) : ((double)(u % nc) + 0.5) * s->lsc - s->hL;
      u /= nc;
      qv[k] = quant8(x[k] - cen, s->qinv);
      Q += qv[k] * qv[k];
    }
    unsigned w[8];
    cand_record<D>(qv, thresh_share(s, sg) - Q, w);
    int4* pp = reinterpret_cast<int4*>(s->qc16 + (size_t)dst * 8);
    pp[0] = make_int4((int)w[0], (int)w[1], (int)w[2], (int)w[3]);
    pp[1] = make_int4((int)w[4], (int)w[5], (int)w[6], (int)w[7]);
  }
  s->oid[pn][dst] = s->ysort ? key & ((1 << 23) - 1) : key;
}

// FIRE 2.0 control for one system (semi-implicit Euler variant, unit masses),
// by one wave: fixed-order reductions of the tile partials, convergence test
// on the current forces, then the P = F.v branch, dt / alpha updates and the
// mixing coefficients.  |v + dt F|^2 is formed from |v|^2, F.v and |F|^2.
__device__ inline FireNext fire_control(const SysDev* s) {
  const int lane = threadIdx.x & 63, nw = s->nwaves;
  double pe = 0, fv = 0, ff = 0, vv = 0, fm = 0;
  const HDMD_GLOBAL double* part = gbl(s->part);
  for (int w = lane; w < nw; w += 64 * 4) {
    double p[4][5];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const HDMD_GLOBAL double* q = part + (size_t)min(w + 64 * u, nw - 1) * kPart;
      p[u][0] = q[P_PE];
      p[u][1] = q[P_FV];
      p[u][2] = q[P_FF];
      p[u][3] = q[P_VV];
      p[u][4] = q[P_FMAX2];
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      if (w + 64 * u >= nw) break;
      pe += p[u][0];
      fv += p[u][1];
      ff += p[u][2];
      vv += p[u][3];
      fm = fmax(fm, p[u][4]);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    pe += __shfl_xor(pe, o, 64);
    fv += __shfl_xor(fv, o, 64);
    ff += __shfl_xor(ff, o, 64);
    vv += __shfl_xor(vv, o, 64);
    fm = fmax(fm, __shfl_xor(fm, o, 64));
  }
  const FireCtl& c = s->fc;
  FireNext r;
  r.pe = pe;
  r.fmax = sqrt(fm);
  r.fdt = s->fdt;
  r.falpha = s->falpha;
  r.c_keep = s->c_keep;
  r.c_mix = s->c_mix;
  r.npos = s->npos;
  r.nneg = s->nneg;
  r.zero = 0;
  r.status = SLOT_DONE;
  r.fstatus = s->fstatus;
  r.err = 0;
  if (!isfinite(pe) || !isfinite(ff)) {
    r.err = ERR_RUN_NAN;
    r.fstatus = -5;
  } else if (sqrt(fm) < c.ftol || (c.etol > 0.0 && pe / (double)s->n < c.etol)) {
    r.fstatus = 0;
  } else if (s->iters >= c.maxiter) {
    r.fstatus = 1;
  } else {
    double dt = s->fdt, alpha = s->falpha;
    bool stop = false;
    if (fv > 0.0) {
      r.npos++;
      r.nneg = 0;
      if (r.npos > c.ndelay) {
        dt = fmin(dt * c.finc, c.dtmax);
        alpha *= c.falpha;
      }
    } else {
      r.npos = 0;
      r.nneg++;
      if (r.nneg > c.nnegmax) {
        stop = true;
      } else {
        if (!(c.initdelay && s->iters < c.ndelay)) {
          if (dt * c.fdec >= c.dtmin) dt *= c.fdec;
          alpha = c.alpha0;
        }
        r.zero = 1;
      }
    }
    if (stop) {
      r.fstatus = 1;
    } else {
      const double v2 = r.zero ? dt * dt * ff : vv + 2.0 * dt * fv + dt * dt * ff;
      const double vn = sqrt(v2), fn = sqrt(ff);
      r.status = SLOT_RUNNING;
      r.fdt = dt;
      r.falpha = alpha;
      r.c_keep = fn > 0.0 ? 1.0 - alpha : 1.0;
      r.c_mix = fn > 0.0 ? alpha * vn / fn : 0.0;
    }
  }
  return r;
}

__device__ inline void fire_commit(SysDev* s, const FireNext& f) {
  s->pe = f.pe;
  s->fmax = f.fmax;
  s->fdt = f.fdt;
  s->falpha = f.falpha;
  s->c_keep = f.c_keep;
  s->c_mix = f.c_mix;
  s->npos = f.npos;
  s->nneg = f.nneg;
  s->c_zero = f.zero;
  s->fstatus = f.fstatus;
  s->err |= f.err;
  if (f.status == SLOT_RUNNING) s->iters++;
  else s->status = f.status;
}

// End of a step / iteration for one system, by one wave: energy reductions
// and thermo row (MD), buffer flips (the permuted buffers after a rebuild,
// otherwise the freshly written position buffer), trigger reset, step counter.
__device__ inline void finalize_system(SysDev* s, bool rb) {
  if (!running(s)) return;
  const int lane = threadIdx.x & 63;
  if (s->err && s->mode != MODE_STATIC && !rb) {
    // the list overflowed after the last finalisation: nothing has run since
    if (lane == 0) s->status = SLOT_DONE;
    return;
  }
  if (s->mode == MODE_MD) {
    const int nw = s->nwaves;
    const bool rec = s->thermo && s->thermo_every > 0 && s->step % s->thermo_every == 0;
    double pe = 0.0, ke = 0.0;
    const HDMD_GLOBAL double* part = gbl(s->part);
    for (int w = lane; w < nw; w += 64 * 8) {
      double a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const size_t o = (size_t)min(w + 64 * u, nw - 1) * kPart;
        a[u] = part[o + P_PE];
        b[u] = part[o + P_KE];
      }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const bool in = w + 64 * u < nw;
        pe += in ? a[u] : 0.0;
        ke += in ? b[u] : 0.0;
      }
    }
    pe = wave_sum(pe);
    ke = wave_sum(ke);
    double vir = 0.0, nc = 0.0, m2 = 0.0, m4 = 0.0, ov = 0.0;
    if (rec) {
      for (int w = lane; w < nw; w += 64) {
        const HDMD_GLOBAL double* pw = part + (size_t)w * kPart;
        vir += pw[P_VIR];
        nc += pw[P_NC];
        m2 += pw[P_M2];
        m4 += pw[P_M4];
        ov += pw[P_OV];
      }
      vir = wave_sum(vir);
      nc = wave_sum(nc);
      m2 = wave_sum(m2);
      m4 = wave_sum(m4);
      ov = wave_sum(ov);
    }
    if (lane == 0) {
      s->pe = pe;
      s->ke = ke;
      if (!isfinite(pe + ke)) s->err |= ERR_RUN_NAN;
      // Berendsen factor for the next full-step kick, from this step's T
      if (s->tau_t > 0.0 && ke > 0.0) {
        const double T = 2.0 * ke / ((double)s->d * (double)(s->n - 1));
        s->vscale = sqrt(1.0 + s->dt / s->tau_t * (s->temp_t / T - 1.0));
      } else {
        s->vscale = 1.0;
      }
      if (rec) {
        double* r = s->thermo + kThermoCols * (s->step / s->thermo_every);
        r[0] = (double)s->step;
        r[1] = ke;
        r[2] = pe;
        r[3] = ke + pe;
        r[4] = vir;                 // sum over pairs of r_ij . F_ij
        r[5] = nc / (double)s->n;   // mean neighbours inside the cutoff (Z)
        // displacement moments since the run's start, alpha_2 (eq. ngp; 0
        // while nothing has moved) and f_ov (eq. fov)
        const double msd = m2 / (double)s->n, mqd = m4 / (double)s->n;
        r[6] = msd;
        r[7] = mqd;
        r[8] = msd > 0.0 ? s->d * mqd / ((s->d + 2) * msd * msd) - 1.0 : 0.0;
        r[9] = ov / (double)s->n;
      }
    }
  }
  if (lane == 0) {
    if (rb) {
      s->pcur ^= 1;
      s->builds++;
    } else {
      s->xcur ^= 1;
    }
    // the shells whose pairs may interact at the new positions
    const double dl = rb ? 0.0 : sqrt(__longlong_as_double((long long)s->maxdisp2));
    s->shells = s->nshell == 1
                    ? 1
                    : 1 + (int)fmin(2.0 * dl * s->sh_scale * (1.0 + 1e-9) + 1e-9, s->nshell - 1.0);
    s->maxdisp2 = 0ull;
    s->force_rebuild = 0;
    if (s->mode == MODE_MD) {
      s->step++;
      if (s->step > s->nsteps) s->status = SLOT_DONE;
    }
    if (s->err) s->status = SLOT_DONE;
  }
}

// Placement of a system alone over grid - 1 workgroups; with a.fin the first
// one finalises the iteration.  The binning has noted whether it rebuilds and
// from which buffers, so that neither the placement nor the list build reads
// what the finalisation changes: an iteration needs no launch of its own for
// it.
template <int D, typename VT>
__global__ __launch_bounds__(256) void k_place(KArgs a) {
  SysDev* s = a.single;
  const bool rb = s->rb != 0;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x == 0) {
    if (a.fin && w == 0) {
      if (a.fin == 2 && live(s) && s->mode == MODE_FIRE) {
        const FireNext f = s->fnext;
        if (threadIdx.x == 0) fire_commit(s, f);
        if (f.status != SLOT_RUNNING) return;
      }
      finalize_system(s, rb);
    }
    return;
  }
  if (!rb) return;
  const int nt = s->ntiles;
  for (int t = (blockIdx.x - 1) * 4 + w; t < nt; t += (gridDim.x - 1) * 4) place_tile<D, VT>(s, t);
}

// ---------------------------------------------------------------------------
// Verlet-list build over the linked subcells (Sec. II.C, Fig. 1)
//
// Linked subcells (n_cell >= 3, and half-size subcells, at least 5 per axis): the
// matrix-core build.  Every atom's offset from its subcell centre is
// quantised to q = y/Delta (Delta = L_sc/250, |q| <= 125), so an atom of the
// subcell o away sits at q_j + 250 o.  A pair is within its list radius
// r_ij = a_i + a_j, a = (c sigma + s)/2, only if |q_j + 250 o - q_i| <
// alpha_i + alpha_j, alpha = a/Delta + sqrt(d)/2 (each axis is off by at most
// one unit), and (alpha_i + alpha_j)^2 <= 2 alpha_i^2 + 2 alpha_j^2 < T_i +
// T_j with T = floor(2 alpha^2) + 1: with q'_i = q_i - 250 o,
//   |q_j - q'_i|^2 < T_i + T_j  <=>  S_ij = q'_i.(2 q_j) + C_j - B'_i > 0,
//   C_j = T_j - |q_j|^2,  B'_i = |q'_i|^2 - T_i.
// S is one entry of a product over 16 f16 slots:
//   candidate [2q_j,d-1, 2048, 1, 1, 2q_j,0 .. 2q_j,d-2, floor(C_j/2048), C_j mod 2048, 0 ..]
//   home      [-q'_i,d-1, floor(B'_i/2048), B'_i mod 2048, 1/2, -q'_i,0 .. -q'_i,d-2, -2048, -1, 0 ..]
// gives 1/2 - S_ij, negative exactly when the pair survives.  Every slot is
// an integer of magnitude <= 2048 or 1/2 (exact in f16: |2q| <= 254, |q'| <=
// 127 + 250 reach, -2^18 < C < 2^18, |B'| < 2^22) and every partial sum is a
// multiple of 1/2 below 2^23 in magnitude, so the f32 accumulation is exact
// in any order.  The subcell shift sits on the home side only: the candidate
// slots are a record of the atom's own, written once by the subcell sort in
// the layout the matrix instruction reads, and the build loads them straight
// into its operands (no conversion, no shuffle); the home slots are remade
// per row of linked subcells, for the home atoms that can reach it.
// Survivors are listed 64 lanes at a time as (home atom, candidate) codes
// and re-tested exactly in FP64 with the per-pair radius -- the operation
// sequence of the list definition -- one per lane; the passing ones are
// appended to their rows.
//
// Bound by VALU and scalar issue: per 256 pair tests one matrix instruction
// and four sign-bit shifts, the rest is row set-up and listing.  Candidates
// as ready operands and word-wise listing replaced per-row conversions,
// operand transposes and a listing walk per home atom (4.4e8 instead of
// 9.3e8 vector instructions per build): d = 6, N = 262144, 64 atoms per
// subcell: 2.14 -> 1.30 ms.  With the rows ordered by shell (below): 1.50; d =
// 6, N = 1e5, 24 per subcell: 1.03 -> 0.56; d = 4, N = 65536, 6.6 per subcell
// (sparse form): 0.43 -> 0.17 ms.
//
// Systems of n_cell <= 2, where several images of a pair can be in reach
// along an axis, and small systems take k_build_wrap below.
// ---------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 hv4 __attribute__((ext_vector_type(4)));
typedef float fv4 __attribute__((ext_vector_type(4)));
typedef unsigned uv2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(4))) const int cint;

// A pointer that is the same in every lane, moved into scalar registers (a
// pointer read from device memory lands in vector registers otherwise).
template <typename T>
__device__ inline T* uniform_ptr(T* p) {
  const unsigned long long u = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
  return reinterpret_cast<T*>(((unsigned long long)hi << 32) | lo);
}

__device__ inline int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline double uniform_dbl(double v) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Orders this wave's LDS writes before its later LDS reads (other lanes).
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The lane-write intrinsic (v_writelane_b32): returns `old` with lane `ln`
// replaced by the uniform `val`.
__device__ int amdgcn_writelane(int val, int ln, int old) __asm("llvm.amdgcn.writelane");

// the lanes below this one whose bit is set in m
__device__ inline int rank_in(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Inclusive prefix sum over the wave's lanes.
__device__ inline int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast 15 to rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast 31 to rows 2, 3
  return v;
}

// One wave's survivors on their way to the exact test.  The sign bits of the
// matrix products come as words of up to 32 bits, most of them zero; the
// others are queued (push), and 64 queued words at a time, one per lane, are
// expanded into codes, one per survivor (expand), so that neither step loops
// over the mostly empty lanes.  Words and codes keep their order: the
// survivors of one home atom come in its candidates' order whatever other
// home atoms share the wave.
constexpr int kWordCap = 192, kCodeCap = 192;
template <typename TAG>
struct SurvivorLds {
  unsigned word[kWordCap];
  unsigned code[kCodeCap];
  TAG tag[kWordCap];
};
template <typename TAG>
struct Survivors {
  SurvivorLds<TAG>* q;
  int nw, nq;

  // queues the lanes' non-zero words (bit 31 - p of a word stands for the
  // code 32 tag + p); the caller sees to it that at most kWordCap - 64 are
  // queued before
  __device__ __attribute__((always_inline)) void push(unsigned w, unsigned tag) {
    const unsigned long long any = __ballot(w != 0u);
    if (w != 0u) {
      const int at = nw + rank_in(any);
      q->word[at] = w;
      q->tag[at] = (TAG)tag;
    }
    nw += __builtin_popcountll(any);
  }
  // expands the first queued words (up to 64) into codes, as many words as
  // the code list has room for; true when it took all of them
  __device__ __attribute__((always_inline)) bool expand(int lane) {
    wave_lds_sync();
    const int n = min(nw, 64);
    unsigned w = lane < n ? q->word[lane] : 0u;
    const unsigned tag = 32u * (unsigned)q->tag[lane];
    const int c = __builtin_popcount(w), e = wave_scan(c);
    const unsigned long long fit = __ballot(lane < n && nq + e <= kCodeCap);
    const int na = __builtin_popcountll(fit);
    if (!((fit >> lane) & 1ull)) w = 0u;
    int at = nq + e - c;
    while (w) {
      const int p = __builtin_clz(w);
      w &= ~(0x80000000u >> p);
      q->code[at++] = tag + p;
    }
    if (na > 0) nq += __builtin_amdgcn_readlane(e, na - 1);
    // the words left move to the front
    const int rest = nw - na;
    unsigned wl[kWordCap / 64];
    TAG tl[kWordCap / 64];
#pragma unroll
    for (int u = 0; u < kWordCap / 64; u++) {
      const int from = min(na + 64 * u + lane, kWordCap - 1);
      wl[u] = q->word[from];
      tl[u] = q->tag[from];
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < kWordCap / 64; u++) {
      if (64 * u + lane < rest) {
        q->word[64 * u + lane] = wl[u];
        q->tag[64 * u + lane] = tl[u];
      }
    }
    nw = rest;
    return na == n;
  }
  // hands the codes to `batch(code, valid)` 64 at a time, one per lane:
  // whole batches only, or, with all, every code and word there is
  template <typename F>
  __device__ __attribute__((always_inline)) void drain(int lane, bool all, F batch) {
    for (;;) {
      wave_lds_sync();
      const bool last = all && nw == 0;
      int t = 0;
      for (; t + 64 <= nq || (last && t < nq); t += 64) {
        const bool valid = t + lane < nq;
        batch(q->code[min(t + lane, kCodeCap - 1)], valid);
      }
      // the codes left move to the front
      const int rest = max(nq - t, 0);
      const unsigned c0 = q->code[min(t + lane, kCodeCap - 1)];
      wave_lds_sync();
      if (lane < rest) q->code[lane] = c0;
      nq = rest;
      if (nw >= 64 || (all && nw > 0)) expand(lane);
      else break;
    }
  }
};

// ---------------------------------------------------------------------------
// Shells.  A listed pair at distance r at the build cannot interact before
// the atoms have moved: its distance shrinks by at most 2 delta while no atom
// is further than delta from its place at the build.  Each row is therefore
// kept in kShells shells of r - r_c, skin/8 wide: shell 0 up to r_c + skin/8,
// and so on.  The force kernels walk the shells that delta has reached
// (m = 1 + floor(16 delta / skin), from the same displacement maximum that
// triggers the rebuild) and leave the rest of the row alone; the pairs they
// skip are beyond the cutoff, so the forces are sums of the same terms.
// Between two builds delta grows from 0 to skin/2, so that a run's steps
// visit (d = 6, r_c = 1.24, skin 0.25) about 65 % of the list on average and
// a single force evaluation after its build 33 %.  The build stamps the
// shell on the entry and, when a wave's rows are complete, orders them by it
// in place (shell_order): they are still in its L2, and the other waves'
// pair tests hide the latency (ordering them in the next force kernel took
// 0.33 ms at d = 6, N = 262144, row 139).  Measured per MD step, whole rows
// and shells: d = 6, N = 262144 FP64 237 and 177 us, mixed 190 and 143 us;
// d = 6, N = 100000 Morse 77 and 59 us; the ordering adds 0.18 ms to the
// 1.30 ms build of the first, 14 builds per 100 steps.
// sh_off covers the rounding of r and of the fixed-point form's coordinates.
// ---------------------------------------------------------------------------
template <typename P>
__device__ inline int shell_entry(P s, int j, double r2, double si, double sj) {
  if (s->nshell == 1) return j;
  // r = r2 / sqrt(r2), a Newton step on the hardware estimate
  double y = __builtin_amdgcn_rsq(r2);
  y = __builtin_fma(y, __builtin_fma(-0.5 * r2 * y, y, 0.5), y);
  const double u = __builtin_fma(r2 * y - s->cutoff * (0.5 * (si + sj)), s->sh_scale, -s->sh_off);
  const int k = r2 > 0.0 ? (int)fmin(fmax(u, 0.0), (double)(kShells - 1)) : 0;
  return j | (k << 28);
}

// Orders rows i0 .. i0 + cnt - 1 (cnt <= 64; row i0 + lane has mylen entries,
// written by this wave) by shell, in place and stably, and writes their shell
// ends.  buf: kShellRow words of LDS.  Rows are taken R at a time (all R fit
// the buffer), 64 / R lanes per row, each on a contiguous piece of at most 32
// entries.  Rows longer than kShellRow keep their order: every shell ends at
// the row's end.
template <typename P>
__device__ __forceinline__ void shell_order(P s, int i0, int cnt, int mylen, int* buf) {
  if (s->nshell == 1) return;
  const int lane = threadIdx.x & 63, npad = s->npad;
  HDMD_GLOBAL int* nl = gbl(s->nl) + i0;
  HDMD_GLOBAL vi4* ends = gbl(reinterpret_cast<vi4*>(s->ends + (size_t)i0 * kShells));
  mylen = lane < cnt ? min(mylen, s->width) : 0;
  const int mx = __builtin_amdgcn_readfirstlane(wave_max_i(mylen));
  if (mx > kShellRow) {
    const int l2 = (int)((unsigned)mylen * 0x10001u);  // (a row may have 65535 entries)
    if (lane < cnt) ends[lane] = vi4{l2, l2, l2, l2};
    return;
  }
  wave_lds_sync();  // the rows are written, the buffer is free
  int lr = 5;  // R = 2^lr rows: at most 32 (two lanes per row)
  while (lr > 0 && mx > (2048 >> lr)) lr--;
  const int R = 1 << lr, S = 64 >> lr;
  for (int r0 = 0; r0 < cnt; r0 += R) {
    const int r = lane & (R - 1), sub = lane >> lr;
    const int len = __shfl(mylen, (r0 + r) & 63);
    const int C = (__builtin_amdgcn_readfirstlane(wave_max_i(len)) + S - 1) >> (6 - lr);
    const int k0 = sub * C;
    unsigned long long in = 0;  // entries per shell, six bits each
    const HDMD_GLOBAL int* src = nl + (size_t)k0 * npad + r0 + r;
    const int m = min(len - k0, C);  // this lane's entries
    // all of the lane's entries in registers: one memory latency per R rows
    int e[32];
#pragma unroll
    for (int k = 0; k < 32; k++) {
      e[k] = -1;
      if (k < m) e[k] = *src;
      src += npad;
    }
#pragma unroll
    for (int k = 0; k < 32; k++) in += k < m ? 1ull << (6 * (e[k] >> 28)) : 0ull;
    // prefix sums over the row's lanes, two shells of 16 bits per word
    unsigned c[4], p[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      c[q] = (unsigned)(in >> (12 * q)) & 63u;
      c[q] |= ((unsigned)(in >> (12 * q + 6)) & 63u) << 16;
      p[q] = c[q];
    }
    for (int o = R; o < 64; o <<= 1) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const unsigned u = __shfl_up(p[q], o);
        if (lane >= o) p[q] += u;
      }
    }
    unsigned end[4], at[4], run = 0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const unsigned t = __shfl(p[q], (S - 1) * R + r);
      // ends of shells 2q, 2q + 1, then the lane's first places in them
      end[q] = (run + (t & 0xffffu)) | ((run + (t & 0xffffu) + (t >> 16)) << 16);
      at[q] = (run | ((run + (t & 0xffffu)) << 16)) + p[q] - c[q];
      run = end[q] >> 16;
    }
#pragma unroll
    for (int k = 0; k < 32; k++) {
      if (k < m) {
        const int sh = e[k] >> 28, sft = (sh & 1) * 16;
        const unsigned w = sh < 4 ? (sh < 2 ? at[0] : at[1]) : (sh < 6 ? at[2] : at[3]);
        buf[(((w >> sft) & 0xffffu) << lr) + r] = e[k];
        const unsigned inc = 1u << sft;
        at[0] += sh < 2 ? inc : 0u;
        at[1] += (sh & ~1) == 2 ? inc : 0u;
        at[2] += (sh & ~1) == 4 ? inc : 0u;
        at[3] += sh >= 6 ? inc : 0u;
      }
    }
    wave_lds_sync();
    for (int k = sub; k < len; k += S) nl[(size_t)k * npad + r0 + r] = buf[(k << lr) + r];
    if (sub == 0 && r0 + r < cnt)
      ends[r0 + r] = vi4{(int)end[0], (int)end[1], (int)end[2], (int)end[3]};
    wave_lds_sync();
  }
}

// Appends a batch's passing pairs to their rows: each sets its bit in its
// home atom's LDS word, whose bits below its own are the pairs before it in
// the batch.  Every lane takes the new length of its own home atoms.
struct RowAppend {
  unsigned long long* hit;  // per home atom
  HDMD_GLOBAL int* nl;
  int npad, W;
  // entry: the row entry of the pair (shell_entry)
  __device__ __attribute__((always_inline)) void operator()(int lane, bool two, bool pass, int h, int i,
                                                            int entry, int& len0, int& len1) const {
    if (pass) atomicOr(hit + h, 1ull << lane);
    const int la = __shfl(len0, h & 63), lb = two ? __shfl(len1, h & 63) : 0;
    wave_lds_sync();
    if (pass) {
      const int pos = (h >= 64 ? lb : la) + rank_in(hit[h]);
      if (pos < W) nl[(size_t)pos * npad + i] = entry;
    }
    len0 += __builtin_popcountll(hit[lane]);
    if (two) len1 += __builtin_popcountll(hit[64 + lane]);
    wave_lds_sync();
    hit[lane] = 0ull;
    if (two) hit[64 + lane] = 0ull;
    wave_lds_sync();
  }
};

// LDS of one wave of the matrix-core build: under 10240 bytes with the 3^d
// stencil, so that 16 such waves share a CU, four per SIMD.
constexpr int kBuildTags = 16;  // segments of candidate blocks the codes may refer to
template <int RAD>
struct BuildLds {  // (at least kShellRow words: shell_order)
  static constexpr int SW = 6 + 2 * (2 * RAD + 1);  // words per staged home atom
  uv2 stage[128 * SW / 2];         // home slots 4..15, then slots 0..3 per last-axis offset
  unsigned long long hit[64 * 2];  // RowAppend
  SurvivorLds<unsigned short> q;
  int base[kBuildTags][16];        // first atom of each candidate block of a segment
  unsigned char hid[128];          // home atom of each compacted column
};

// One home subcell of a system that rebuilds, split over G waves: gw (< G)
// selects this wave's share of the home atoms.
//
// A row is the 2 RAD + 1 linked subcells along the last axis.  BUILD_DENSE
// (more than 16 atoms per subcell on average): a segment is one row's
// candidates in blocks of 16, up to NB per subcell, all held in registers
// while the kept home atoms of the row (compacted into columns) pass over
// them 16 at a time.  BUILD_SPARSE (the 3^d stencil): a segment is the rows along the last
// two axes, one block of each of their 9 subcells, against all home atoms of
// a pass of up to 40, so that their loads are in flight together.
template <int D, int RAD, int MODE>
struct BuildTile {
  static constexpr bool DENSE = MODE != BUILD_SPARSE;
  static_assert(RAD == 1 || MODE == BUILD_DENSE, "half-size subcells take the dense form");
  static constexpr int NRS = 2 * RAD + 1;
  static constexpr int SW = BuildLds<RAD>::SW;
  static constexpr int NR = DENSE ? 1 : NRS;       // rows per segment
  static constexpr int NB = DENSE ? 15 / NRS : 1;  // blocks per subcell and segment
  static constexpr int NT = NR * NRS * NB;         // blocks per segment (at most 15)
  static constexpr int NW = (D + 4) / 2 - 1;       // packed words of slots 4 .. d+4
  static constexpr int HP = DENSE ? 128 : 40;      // home atoms per pass

  cSys* s;
  BuildLds<RAD>* m;
  cint* flat;
  const int* rec;
  const double* xb;
  HDMD_GLOBAL int* nl;
  double L, invL, cut, skin;
  int nc, npad, W, hb, hcnt, lane;
  int ci[D], stride[D];
  bool two, v0, v1;
  Survivors<unsigned short> sv;
  int ntag;                    // segments tagged
  int len0, len1;      // row lengths of the lane's home atoms
  unsigned hn0[NW], hn1[NW];   // packed f16 slots 4 .. d+4 at offset zero
  float ql0, ql1, B0, B1, tc0, tc1;

  // home slots of slot word t at outer offsets `oa` (packed 250 o)
  __device__ __attribute__((always_inline)) void put_home(const unsigned (&hn)[NW], float ql, float B,
                                                          const unsigned (&oa)[NW], int osq, int slot) {
    uv2* e = m->stage + slot * (SW / 2);
    unsigned w[6];
    float sB = 0.0f;
#pragma unroll
    for (int t = 0; t < 6; t++) {
      w[t] = 0u;
      if (t < NW) {
        // -q' = -q + 250 o;  sum of 250 o (-q) for B'
        w[t] = h2u(u2h(hn[t]) + u2h(oa[t]));
        sB = __builtin_amdgcn_fdot2(u2h(hn[t]), u2h(oa[t]), sB, false);
      }
    }
    e[0] = uv2{w[0], w[1]};
    e[1] = uv2{w[2], w[3]};
    e[2] = uv2{w[4], w[5]};
    const float Bo = B + 2.0f * sB + (float)(kQScale * kQScale) * (float)osq;
#pragma unroll
    for (int r = 0; r < NRS; r++) {
      const float sh = (float)(kQScale * (r - RAD));
      const float b = Bo + 2.0f * sh * ql + sh * sh;
      const float hi = floorf(b * (1.0f / 2048.0f)), lo = __builtin_fmaf(-2048.0f, hi, b);
      e[3 + r] = uv2{__builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(ql + sh, hi)),
                     __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(lo, 0.5f))};
    }
  }

  // squared gap of the lane's home atoms to the subcells o away along axis k
  // (one unit short), added to S
  __device__ __attribute__((always_inline)) void add_gap(int k, int o, float& S0, float& S1) const {
    if (o == 0) return;
    const float face = (float)((kQScale / 2) * (2 * (o < 0 ? -o : o) - 1) - 1);
    const float sg = o < 0 ? -1.0f : 1.0f;
    const float a0 = (float)u2h(hn0[k / 2])[k % 2], a1 = (float)u2h(hn1[k / 2])[k % 2];
    const float g0 = fmaxf(__builtin_fmaf(sg, a0, face), 0.0f);
    const float g1 = fmaxf(__builtin_fmaf(sg, a1, face), 0.0f);
    S0 = __builtin_fmaf(g0, g0, S0);
    S1 = __builtin_fmaf(g1, g1, S1);
  }

  __device__ __attribute__((always_inline)) int wrapc(int c) const {
    return c < 0 ? c + nc : (c >= nc ? c - nc : c);
  }
  // packed 250 o of axis k added to the offset words
  __device__ __attribute__((always_inline)) static unsigned off_word(int k, int o) {
    // f16 250 = 0x5bd0, 500 = 0x5fd0
    const unsigned a = o == 0 ? 0u : ((o == 1 || o == -1) ? 0x5bd0u : 0x5fd0u) | (o < 0 ? 0x8000u : 0u);
    return a << (16 * (k % 2));
  }

  // exact test of the listed survivors, one per lane
  __device__ __attribute__((always_inline)) void drain(bool all) {
    const RowAppend append{m->hit, nl, npad, W};
    sv.drain(lane, all, [&](unsigned cd, bool valid) {
      // code: home atom, segment, lane group, position (4 block + row)
      const int h = valid ? (int)(cd >> 12) : 0, i = hb + h;
      int j = m->base[(cd >> 8) & 15][(cd >> 2) & 15] + 4 * ((cd >> 6) & 3) + (cd & 3);
      j = valid ? j : i;
      double xi[D], si, xj[D], sj;
      load_rec<D>(xb, i, xi, si);
      load_rec<D>(xb, j, xj, sj);
      // The nearest image is taken with rint: the radius is at most L/3 (on
      // half-size subcells, at least 5 per axis: 2L/5), so every pair it can
      // admit has all |dx_k| clear of L/2, where rint and the definition's
      // shift give the same value bit for bit; pairs with some |dx_k| near
      // L/2 are beyond the radius either way.
      double r2 = 0.0;
#pragma unroll
      for (int k = 0; k < D; k++) {
        const double dx = near_image(xj[k] - xi[k], L, invL);
        r2 = __builtin_fma(dx, dx, r2);
        __builtin_amdgcn_sched_barrier(0);  // one axis at a time: few live registers
      }
      const bool pass = j != i && r2 < list_r2(si, sj, cut, skin);
      append(lane, two, pass, h, i, shell_entry(s, j, r2, si, sj), len0, len1);
    });
    if (all) ntag = 0;
  }

  // the candidate blocks of one segment (each subcell's atoms from k0 on)
  // against the staged home columns of its rows (ncol columns, st apart).
  // Block t = k NR NRS + r is the k-th of subcell r.
  __device__ __attribute__((always_inline)) void segment(const int (&f0)[NR * NRS],
                                                         const int (&f1)[NR * NRS], unsigned rows,
                                                         int k0, int kn, int ncol, int st) {
    constexpr int NS = NR * NRS;
    const int g = lane >> 4, col = lane & 15;
    const int nhb = (ncol + 15) >> 4;
    int b0 = 0;
    for (;;) {
      hv4 X[NT];
#pragma unroll
      for (int k = 0; k < NB; k++) {
        if (k > 0 && k >= kn) continue;
#pragma unroll
        for (int r = 0; r < NS; r++) {
          const int a = f0[r] + k0;
          int n = max(f1[r] - a, 0);
          if (!DENSE) n = (rows >> (r / NRS)) & 1u ? n : 0;
          // loads past the subcell's end give zero slots, which never pass
          const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(rec + (size_t)a * 8), 0, n * 32,
                                                            0x00020000);
          X[k * NS + r] = __builtin_bit_cast(
              hv4, __builtin_amdgcn_raw_buffer_load_b64(rs, col * 32 + g * 8 + k * 512, 0, 0));
        }
      }
      {  // where the codes of this segment find their atoms
        int b;
        if constexpr (DENSE) {
          const int r = lane % NRS;
          b = f0[0];
#pragma unroll
          for (int q = 1; q < NRS; q++) b = r == q ? f0[q] : b;
          b += k0 + 16 * (lane / NRS);
        } else {
          b = 0;
#pragma unroll
          for (int r = 0; r < NS; r++) b = amdgcn_writelane(f0[r] + k0, r, b);
        }
        if (lane < 16) m->base[ntag][lane] = b;
      }
      bool full = false;
      for (; b0 < nhb && !full; b0++) {
        const int hs = 16 * b0 + col;
        hv4 H[NS];
#pragma unroll
        for (int u = 0; u < NR; u++)
#pragma unroll
          for (int r = 0; r < NRS; r++)
            H[u * NRS + r] = __builtin_bit_cast(
                hv4, m->stage[(st * u + hs) * (SW / 2) + (g == 0 ? 3 + r : g - 1)]);
        unsigned w0 = 0u, w1 = 0u;
#pragma unroll
        for (int k = 0; k < NB; k++) {
          // (levels beyond the longest subcell: their bits are zero)
          if (k > 0 && k >= kn) {
#pragma unroll
            for (int r = 0; r < NS; r++) {
              if (k * NS + r < 8) w0 <<= 4;
              else w1 <<= 4;
            }
            continue;
          }
          // a row's products at a time, their results packed before the next
          // row's (few live registers)
#pragma unroll
          for (int u = 0; u < NR; u++) {
            if (!DENSE && !((rows >> u) & 1u)) {
              // no home atom reaches the row: its columns were not staged
#pragma unroll
              for (int r = 0; r < NRS; r++) {
                if (k * NS + u * NRS + r < 8) w0 <<= 4;
                else w1 <<= 4;
              }
              continue;
            }
            fv4 e[NRS];
#pragma unroll
            for (int r = 0; r < NRS; r++) {
              const fv4 zero = {};
              const int t = k * NS + u * NRS + r;
              e[r] = __builtin_amdgcn_mfma_f32_16x16x16f16(X[t], H[u * NRS + r], zero, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < NRS; r++) {
              unsigned& w = k * NS + u * NRS + r < 8 ? w0 : w1;
#pragma unroll
              for (int v = 0; v < 4; v++)
                w = __builtin_amdgcn_alignbit(w, __float_as_uint(e[r][v]), 31u);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        static_assert(NT > 8 && NT <= 16, "two words of bits");
        w1 <<= 4 * (16 - NT);
        // columns past the last home atom hold whatever the stage held
        const bool hv = hs < ncol;
        const int h = DENSE ? (int)m->hid[hs] : hs;
        const unsigned tag = (unsigned)((h << 7) | (ntag << 3) | (g << 1));
        sv.push(hv ? w0 : 0u, tag);
        if (!DENSE || kn * NS > 8) sv.push(hv ? w1 : 0u, tag | 1u);
        while (sv.nw >= 64 && !full) full = !sv.expand(lane);
      }
      const bool done = b0 >= nhb;
      if (done) ntag++;
      // the exact test runs outside the blocks' register lifetime: a segment
      // it interrupts loads them again
      if (full || sv.nq >= 128 || ntag == kBuildTags) drain(ntag == kBuildTags);
      if (done) break;
    }
  }

  // one segment's rows: subcell bounds, staging, and the walk over subcells
  // longer than a segment
  __device__ __attribute__((always_inline)) void rows_at(float S0, float S1, int P,
                                                         const unsigned (&oa)[NW], int osq) {
    int f0[NR * NRS], f1[NR * NRS];
    unsigned rows = 0;
    unsigned long long km0 = 0, km1 = 0;
    int mx = 0;
#pragma unroll
    for (int u = 0; u < NR; u++) {
      int Pu = P;
      if (!DENSE) Pu += wrapc(ci[D - 2] + u - RAD) * nc;
#pragma unroll
      for (int r = 0; r < NRS; r++) {
        const int c = Pu + wrapc(ci[D - 1] + r - RAD);
        f0[u * NRS + r] = flat[c];
        f1[u * NRS + r] = flat[c + 1];
      }
    }
    wave_lds_sync();  // the previous rows' columns have been read
    int ncol = 0, st = 0;
    if (DENSE) {
      km0 = __ballot(v0 && S0 < tc0);
      km1 = two ? __ballot(v1 && S1 < tc1) : 0ull;
      const int nk0 = __builtin_popcountll(km0);
      ncol = nk0 + __builtin_popcountll(km1);
      if ((km0 >> lane) & 1ull) {
        const int r = rank_in(km0);
        m->hid[r] = (unsigned char)lane;
        put_home(hn0, ql0, B0, oa, osq, r);
      }
      if (km1 && ((km1 >> lane) & 1ull)) {
        const int r = nk0 + rank_in(km1);
        m->hid[r] = (unsigned char)(64 + lane);
        put_home(hn1, ql1, B1, oa, osq, r);
      }
      rows = 1u;
    } else {
      ncol = hcnt;
      st = hcnt;
#pragma unroll
      for (int u = 0; u < NR; u++) {
        const int o = u - RAD;
        float T0 = S0, T1 = S1;
        add_gap(D - 2, o, T0, T1);
        if (__ballot(v0 && T0 < tc0) == 0ull) continue;
        rows |= 1u << u;
        if (v0) {
          unsigned ou[NW];
#pragma unroll
          for (int t = 0; t < NW; t++) ou[t] = oa[t];
          ou[(D - 2) / 2] |= off_word(D - 2, o);
          put_home(hn0, ql0, B0, ou, osq + o * o, u * hcnt + lane);
        }
      }
      if (!rows) return;
    }
#pragma unroll
    for (int r = 0; r < NR * NRS; r++) mx = max(mx, f1[r] - f0[r]);
    wave_lds_sync();
    for (int k0 = 0; k0 < mx; k0 += 16 * NB)
      segment(f0, f1, rows, k0, min((mx - k0 + 15) >> 4, NB), ncol, st);
  }

  // outer offsets of axis K and beyond (in stencil order, last axis fastest),
  // leaving out those that no home atom reaches
  template <int K>
  __device__ __attribute__((always_inline)) void walk(float S0, float S1, int P, const unsigned (&oa)[NW],
                                                      int osq) {
    if constexpr (K >= (DENSE ? D - 1 : D - 2)) {
      rows_at(S0, S1, P, oa, osq);
    } else {
#pragma unroll 1
      for (int o = -RAD; o <= RAD; o++) {
        // A SIMD issues for its oldest waves first, so that without this the
        // waves of a launch finish one by one and the last ones run alone,
        // their latencies exposed.  A wave's priority falls as it gets
        // through its rows: those that lag get the issue slots.
        if constexpr (K == 0) {
          if (o == -RAD) __builtin_amdgcn_s_setprio(2);
          else if (o == 0) __builtin_amdgcn_s_setprio(1);
          else if (o == RAD) __builtin_amdgcn_s_setprio(0);
        }
        float T0 = S0, T1 = S1;
        add_gap(K, o, T0, T1);
        if (__ballot((v0 && T0 < tc0) || (v1 && T1 < tc1)) == 0ull) continue;
        unsigned ob[NW];
#pragma unroll
        for (int t = 0; t < NW; t++) ob[t] = oa[t] | (t == K / 2 ? off_word(K, o) : 0u);
        walk<K + 1>(T0, T1, P + wrapc(ci[K] + o) * stride[K], ob, osq + o * o);
      }
    }
  }

  // the lane's home atom of slot ii: its own candidate record turned into
  // home slots at offset zero, and its reach for the row cull: its share of
  // the radius plus half the largest, a_i + r_l,max/2
  __device__ __attribute__((always_inline)) void own(int ii, unsigned (&hn)[NW], float& ql, float& B,
                                                     float& tc) const {
    const v4i a = *reinterpret_cast<const v4i*>(rec + (size_t)ii * 8);
    const v4i b = *reinterpret_cast<const v4i*>(rec + (size_t)ii * 8 + 4);
    const unsigned w[8] = {(unsigned)a.x, (unsigned)a.y, (unsigned)a.z, (unsigned)a.w,
                           (unsigned)b.x, (unsigned)b.y, (unsigned)b.z, (unsigned)b.w};
    auto slot = [&](int k) { return u2h(w[k / 2])[k % 2]; };
    ql = -0.5f * (float)slot(0);
    B = -__builtin_fmaf(2048.0f, (float)slot(D + 3), (float)slot(D + 4));
#pragma unroll
    for (int t = 0; t < NW; t++) {
      hv2 v;
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const int k = 4 + 2 * t + e;
        v[e] = k < D + 3 ? (_Float16)-0.5f * slot(k)
                         : (k == D + 3 ? (_Float16)-2048.0f : (k == D + 4 ? (_Float16)-1.0f : (_Float16)0.0f));
      }
      hn[t] = h2u(v);
    }
    const double sg = xb[(size_t)ii * Dims<D>::DR + D];
    const double reach = (0.5 * (cut * sg + skin) + 0.5 * s->rlmax) * s->qinv;
    tc = (float)ceil(reach * reach);
  }

  __device__ __attribute__((always_inline)) void run(SysDev* sys, int hc, int gw, int G, BuildLds<RAD>* lds) {
    s = (cSys*)sys;
    m = lds;
    lane = threadIdx.x & 63;
    // subcell starts come through the scalar cache (written by an earlier kernel)
    flat = (cint*)s->cell_flat;
    const int c0h = flat[hc], c1h = flat[hc + 1];
    const int per = (c1h - c0h + G - 1) / G;
    const int h0 = c0h + gw * per, h1 = min(c1h, h0 + per);
    if (h0 >= h1) return;
    nc = s->ncell;
    npad = s->npad;
    W = s->width;
    xb = s->x[s->rx];
    rec = s->qc16;
    nl = gbl(s->nl);
    L = s->L;
    invL = 1.0 / L;
    cut = s->cutoff;
    skin = s->skin;
    {
      int u = hc, sd = 1;
#pragma unroll
      for (int k = D - 1; k >= 0; k--) {
        ci[k] = u % nc;
        u /= nc;
        stride[k] = sd;
        sd *= nc;
      }
    }
    int rowmax = 0;
    // home atoms in passes of up to HP: lane l holds atoms hb + l and hb + 64 + l
    for (hb = h0; hb < h1; hb += HP) {
      hcnt = min(HP, h1 - hb);
      two = DENSE && hcnt > 64;
      v0 = lane < hcnt;
      v1 = two && lane + 64 < hcnt;
      own(v0 ? hb + lane : hb, hn0, ql0, B0, tc0);
      own(v1 ? hb + 64 + lane : hb, hn1, ql1, B1, tc1);
      len0 = len1 = 0;
      sv.q = &m->q;
      sv.nw = sv.nq = 0;
      ntag = 0;
      m->hit[lane] = 0ull;
      m->hit[64 + lane] = 0ull;
      unsigned oa[NW];
#pragma unroll
      for (int t = 0; t < NW; t++) oa[t] = 0u;
      walk<0>(0.0f, 0.0f, 0, oa, 0);
      drain(true);
#pragma unroll 1
      for (int set = 0; set < (two ? 2 : 1); set++)
        shell_order(s, hb + 64 * set, min(hcnt - 64 * set, 64), set ? len1 : len0,
                    reinterpret_cast<int*>(m));
      if (v0) {
        gbl(s->nlen)[hb + lane] = len0;
        rowmax = max(rowmax, len0);
      }
      if (v1) {
        gbl(s->nlen)[hb + 64 + lane] = len1;
        rowmax = max(rowmax, len1);
      }
    }
    rowmax = wave_max_i(rowmax);
    if (lane == 0 && rowmax > 0) {
      atomicMax(&sys->max_row, rowmax);
      if (rowmax > W) atomicOr(&sys->err, ERR_OVERFLOW);
    }
  }
};

template <int D, int RAD, int MODE>
__device__ __forceinline__ void build_mf_tile(SysDev* s, int hc, int gw, int G, BuildLds<RAD>* lds) {
  BuildTile<D, RAD, MODE> t;
  t.run(s, hc, gw, G, lds);
}

template <int D, int G, int RAD, int MODE>
__global__ __launch_bounds__(64 * G, 4) void k_build_mf(KArgs a) {
  __shared__ BuildLds<RAD> lds[G];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int t = xcd_tile(blockIdx.x, gridDim.x);; t += gridDim.x) {
    SysDev* s;
    int hc;
    if (!fetch_cell_tile_u(a, t, s, hc)) break;
    cSys* c = (cSys*)s;
    if (!rebuilding(a, c) | (c->reach != RAD) | (c->wrap != 0) | (c->bmode != MODE)) {
      if (a.single) break;  // one system: the same for every tile
      continue;
    }
    build_mf_tile<D, RAD, MODE>(s, hc, wv, G, &lds[wv]);
  }
}

// ---------------------------------------------------------------------------
// Verlet-list build of systems of n_cell <= 2 (a list radius of a third of
// the box or more) and of small systems: every atom is a candidate of every
// other, and the pair test runs on the matrix cores too.  Along each axis the atom is put on the
// circle, e = (cos, sin)(2 pi x / L): the chord between two atoms does not
// exceed the arc, so a pair within its radius r_ij = a_i + a_j has
//   sum_k |e_i - e_j|_k^2 <= (2 pi r_ij / L)^2
//   <=>  sum_k e_i.e_j >= d - (2 pi r_ij / L)^2 / 2,
// whatever images the periodic box takes, and (a_i + a_j)^2 <= 2 a_i^2 + 2
// a_j^2 splits the bound into a share t = d/2 - (2 pi a / L)^2 (minus a margin
// for the f16 rounding) per atom:
//   t_i + t_j - sum_k e_i.e_j < 0
// is one entry of a product over 2 d + 2 f16 slots
//   candidate [cos, sin of every axis, 1, t_j, 0 ..],  home [-cos, -sin, t_i, 1, 0 ..].
// (The chord test keeps about twice the pairs of the list in d = 8; it takes
// no row cull, no shifts and no wrapped differences.)  2 d + 2 <= 16 (d <=
// 7): records of 16 slots and 16x16x16 products; above: 24 slots, 16x16x32.
// A wave takes up to 16 HB home atoms (HB = 4: a tile; HB = 1: 16 or, in lone
// systems of long rows, 4) as HB blocks of columns held in registers
// and streams all atoms past them, 128 at a time: for a tile 32
// matrix instructions and 128 sign-bit shifts per 8192 pair tests, and the
// exact tests of the survivors.  The survivors of a row come in the order of
// the candidates whatever HB is, so every HB gives the same rows.
// d = 8, N = 131072 (mean row 200): 2.4 ms, where packed int16 tests of the
// 45 % of the pairs that a row cull left took 7.6.
// ---------------------------------------------------------------------------
struct WrapLds {
  unsigned long long hit[64];
  SurvivorLds<unsigned> q;
  int pad[kShellRow - 128 - sizeof(SurvivorLds<unsigned>) / 4];  // shell_order takes it all
};

// Home atoms hb .. hb + homes - 1 (homes <= 16 HB).
template <int D, int HB>
__device__ __forceinline__ void build_wrap_tile(SysDev* sys, int hb, int homes, WrapLds* m) {
  typedef WrapRec<D> R;
  typedef typename std::conditional<R::LW == 2, hv4, hv8>::type Op;
  cSys* s = (cSys*)sys;
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int n = s->n, npad = s->npad, W = s->width;
  if (hb >= n) return;
  const int hcnt = min(homes, n - hb);
  const double* __restrict__ xb = s->x[s->rx];
  const int* __restrict__ rec = s->qc16;
  const double L = s->L, hL = s->hL, cut = s->cutoff, skin = s->skin;
  // operand words of the atom `a + col` (zero past `cnt` atoms, which gives
  // an entry of t_i + 0 or 0: masked by the caller for homes, and never
  // negative for candidates, whose slots are all zero)
  auto operand = [&](int a, int cnt) __attribute__((always_inline)) -> Op {
    const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(rec + (size_t)a * R::WORDS), 0,
                                                      max(min(cnt, 16), 0) * R::WORDS * 4, 0x00020000);
    if constexpr (R::LW == 2) {
      return __builtin_bit_cast(Op, __builtin_amdgcn_raw_buffer_load_b64(rs, col * 32 + g * 8, 0, 0));
    } else {
      // 24 slots: the fourth lane group's eight are zero (out of range)
      const int off = g < 3 ? col * 48 + g * 16 : 16 * 48;
      return __builtin_bit_cast(Op, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    }
  };
  Op H[HB];
#pragma unroll
  for (int b = 0; b < HB; b++) {
    // home slots from the atom's record: signs flipped, 1 and t exchanged
    Op h = operand(hb + 16 * b, hcnt - 16 * b);
    constexpr int GS = R::LW * 2;             // slots per lane group
    constexpr int PG = 2 * D / GS, PS = 2 * D % GS;  // group and place of the slots (1, t)
#pragma unroll
    for (int e = 0; e < GS; e++) H[b][e] = -h[e];
    if (g == PG) {
      H[b][PS] = h[PS + 1];
      H[b][PS + 1] = h[PS];
    }
  }
  Survivors<unsigned> sv{&m->q, 0, 0};
  m->hit[lane] = 0ull;
  const RowAppend append{m->hit, gbl(s->nl), npad, W};
  int len0 = 0, len1 = 0;
  constexpr int SPAN = 1 << 26;  // candidates a code can name
  for (int c0 = 0; c0 < n; c0 += SPAN) {
    const int ce = min(n - c0, SPAN);
    auto drain = [&](bool all) __attribute__((always_inline)) {
      sv.drain(lane, all, [&](unsigned cd, bool valid) {
        // code: pair of chunks, home atom, lane group, position (4 block + row)
        const int h = valid ? (int)(cd >> 7) & 63 : 0, i = hb + h, p = cd & 31;
        int j = c0 + (int)(cd >> 13) * 128 + 16 * (p >> 2) + 4 * ((cd >> 5) & 3) + (p & 3);
        // (j < n but for a home atom whose coordinates are not finite)
        j = valid && j < n ? j : i;
        double xi[D], si, xj[D], sj;
        load_rec<D>(xb, i, xi, si);
        load_rec<D>(xb, j, xj, sj);
        const double r2 = dist2_exact<D>(xi, xj, L, hL);
        const bool pass = j != i && r2 < list_r2(si, sj, cut, skin);
        append(lane, false, pass, h, i, shell_entry(s, j, r2, si, sj), len0, len1);
      });
    };
    // the next 64 candidates' operands are on their way while these are used
    Op X[4], Y[4];
    auto fetch = [&](int a0, Op(&Z)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < 4; b++) {
        const int a = a0 + 16 * b;
        Z[b] = operand(c0 + min(a, ce), ce - a);
      }
    };
    fetch(0, X);
    for (int c = 0; c < ce; c += 128) {
      unsigned w[HB];
#pragma unroll
      for (int h = 0; h < HB; h++) w[h] = 0u;
#pragma unroll
      for (int half = 0; half < 2; half++) {
        fetch(c + 64 * half + 64, half ? X : Y);
#pragma unroll
        for (int b = 0; b < 4; b++) {
          const Op& x = half ? Y[b] : X[b];
          fv4 e[HB];
#pragma unroll
          for (int h = 0; h < HB; h++) {
            const fv4 zero = {};
            if constexpr (R::LW == 2) e[h] = __builtin_amdgcn_mfma_f32_16x16x16f16(x, H[h], zero, 0, 0, 0);
            else e[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, H[h], zero, 0, 0, 0);
          }
#pragma unroll
          for (int h = 0; h < HB; h++)
#pragma unroll
            for (int v = 0; v < 4; v++)
              w[h] = __builtin_amdgcn_alignbit(w[h], __float_as_uint(e[h][v]), 31u);
          if (HB > 1) __builtin_amdgcn_sched_barrier(0);  // one block's results at a time
        }
      }
#pragma unroll 1
      for (int h = 0; h < HB; h++) {
        const int hs = 16 * h + col;
        unsigned wh = w[0];
        if constexpr (HB == 4) wh = h < 2 ? (h == 0 ? w[0] : w[1]) : (h == 2 ? w[2] : w[3]);
        sv.push(hs < hcnt ? wh : 0u, (unsigned)(((c >> 7) << 8) | (hs << 2) | g));
        bool full = false;
        while (sv.nw >= 64 && !full) full = !sv.expand(lane);
        if (full || sv.nq >= 128) drain(false);
      }
    }
    drain(true);
  }
  shell_order(s, hb, hcnt, len0, reinterpret_cast<int*>(m));
  int rowmax = 0;
  if (lane < hcnt) {
    gbl(s->nlen)[hb + lane] = len0;
    rowmax = len0;
  }
  rowmax = wave_max_i(rowmax);
  if (lane == 0 && rowmax > 0) {
    atomicMax(&sys->max_row, rowmax);
    if (rowmax > W) atomicOr(&sys->err, ERR_OVERFLOW);
  }
}

// One system: a tile per workgroup, or (HB = 1) `few` (4 or 16) atoms of one.
template <int D, int HB>
__global__ __launch_bounds__(64, 4) void k_build_wrap(KArgs a, int few) {
  __shared__ WrapLds lds;
  const int homes = HB == 1 ? few : 16 * HB, per = kTile / homes;  // workgroups per tile
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile_u(a, t / per, s, tile)) break;
    cSys* c = (cSys*)s;
    if (!rebuilding(a, c) | (c->wrap == 0)) {
      if (a.single) break;  // one system: the same for every tile
      continue;
    }
    build_wrap_tile<D, HB>(s, tile * kTile + t % per * homes, homes, &lds);
  }
}

// ---------------------------------------------------------------------------
// pair forces over one Verlet row (Sec. II.B getforce)
// ---------------------------------------------------------------------------
// F_i = sum_j fc (x_i - x_j) with fc = -U'(r)/r for r < c sigma_ij;
// e_i = 1/2 sum_j U(r).
// 1/x from the hardware reciprocal estimate and two Newton-Raphson steps
// (each squares the relative error): within an ulp or two of 1/x.
__device__ inline double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return r;
}

// 1/sqrt(x) from the hardware estimate and two Newton-Raphson steps
// y <- y (3/2 - x y^2 / 2).
__device__ inline double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = __builtin_fma(y, __builtin_fma(-hx * y, y, 0.5), y);
  y = __builtin_fma(y, __builtin_fma(-hx * y, y, 0.5), y);
  return y;
}

// MORSE selects the truncated, shifted Morse form at compile time: its
// exponential needs registers that would otherwise count against every force
// loop (WCA and harmonic share the other instantiation, switched at run time).
template <bool MORSE>
__device__ inline void pair_f64(int pot, double eps, double ma, double r2, double sij, double& fc,
                                double& u) {
  if constexpr (MORSE) {  // truncated, shifted Morse (Sec. II.A, eq. morsepot)
    // with t = e^{-a(r - sigma)}: U = eps (t - 1)^2, -U'(r)/r = 2 a eps t (t - 1) / r
    const double ir = rsqrt_nr(r2);  // 1/r
    const double t = exp(-ma * (r2 * ir - sij));
    fc = 2.0 * ma * eps * t * (t - 1.0) * ir;
    u = eps * (t - 1.0) * (t - 1.0);
    (void)pot;
  } else if (pot == 0) {  // WCA
    const double inv = recip(r2);
    const double s2 = sij * sij * inv;
    const double s6 = s2 * s2 * s2;
    fc = 24.0 * eps * (2.0 * s6 * s6 - s6) * inv;
    u = 4.0 * eps * (s6 * s6 - s6) + eps;
  } else {         // harmonic soft spheres
    const double ir = rsqrt_nr(r2);  // 1/r
    const double is = recip(sij);
    const double g = 1.0 - (r2 * ir) * is;
    fc = eps * g * is * ir;
    u = 0.5 * eps * g * g;
  }
}

// SWAP Monte Carlo (Sec. II.D).  Attempt k exchanges the diameters of the
// atoms with caller ids pairs[2k] and pairs[2k+1]; the energies before and
// after (eq. ebefore) sum the pair terms of both atoms with every partner
// inside the cutoff; the pair of the two atoms keeps its diameter and
// cancels.  Kept on the Metropolis rule dE <= 0 or u_k < exp(-dE/T).
// The attempts keep their serial meaning (each sees the diameters the
// earlier ones left) but run in batches: every attempt of a batch gets its
// dE from the diameters at the batch's start (one workgroup each), then one
// workgroup walks the batch in order and settles an attempt unless an
// earlier attempt of the batch that was kept or put off involves an atom
// within the interaction range c sigma_max of one of its atoms (then its dE
// could differ: it is put off to the next batch, ahead of the unbatched
// ones).  Settled attempts commute with the put-off ones they do not touch,
// so the outcome is that of the serial walk.  Diameters live in the records
// (read past the L1, as a kept swap rewrites them) and in diam (caller
// order).
__device__ inline double sig_get(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void sig_put(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// dE of exchanging the diameters of the atoms in slots pi and pj, with the
// current diameters, by a whole workgroup of up to 16 waves: the linked
// subcells of each atom's subcell (all subcells when n_cell <= 2) in groups
// of 64 per wave (a group's bounds loaded by its lanes at once), the lanes
// striding over the group's atoms, the wave sums added in wave order.  Every
// thread returns the same value.  Bound by the latency of a wave's loads: a
// subcell holds a few atoms only, so a lane finds its atom among those of the
// whole group (a search in the prefix sums of the counts) instead of the
// wave taking one subcell after the other (d = 6, N = 100000, 729 subcells
// of 6.4 atoms, 256 attempts: 105 -> 58 us).
template <int D>
__device__ inline double swap_de(const SysDev* s, int pi, int pj, double (*red)[16], double& si_out,
                                 double& sj_out) {
  constexpr int DR = Dims<D>::DR;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
  const int nc = s->ncell;
  const double L = s->L, h = s->hL, cut = s->cutoff, eps = s->eps, ma = s->morse_a;
  const int pot = s->potential;
  const bool morse = pot == kPotMorse;
  double* xb = s->x[s->xcur];
  const int* flat = s->cell_flat;
  // the linked subcells: offsets -reach..+reach per axis, or every subcell
  // once where an axis has fewer than 2 reach + 1
  const int reach = s->reach, rx = nc < 2 * reach + 1 ? nc : 2 * reach + 1;
  const bool dedup = nc < 2 * reach + 1;
  int nst = 1;
  for (int k = 0; k < D; k++) nst *= rx;
  const double si = sig_get(xb + (size_t)pi * DR + D), sj = sig_get(xb + (size_t)pj * DR + D);
  si_out = si;
  sj_out = sj;
  const double far = cut * 0.5 * (fmax(si, sj) + s->sigma_max), far2 = far * far * (1.0 + 1e-12);
  double eb = 0.0, ea = 0.0;
  if (pi != pj) {
    for (int side = 0; side < 2; side++) {
      const int p = side ? pj : pi, o = side ? pi : pj;
      const double sa = side ? sj : si, sb = side ? si : sj;  // p's diameter before, after
      double xp[D];
      load_x<D>(xb, p, xp);
      int cd[D];
      {
        int r = flat_cell<D>(s, xp);
        for (int a = D - 1; a >= 0; a--) {
          cd[a] = r % nc;
          r /= nc;
        }
      }
      for (int t0 = wv * 64; t0 < nst; t0 += 64 * nwv) {
        int cs = 0, ce = 0;
        const int t = t0 + lane;
        if (t < nst) {
          int cell = 0, r = t, mult = 1;
          for (int a = D - 1; a >= 0; a--) {
            int ca;
            if (dedup) {
              ca = r % nc;
              r /= nc;
            } else {
              ca = cd[a] + r % rx - reach;
              r /= rx;
              ca = ca < 0 ? ca + nc : (ca >= nc ? ca - nc : ca);
            }
            cell += ca * mult;
            mult *= nc;
          }
          cs = flat[cell];
          ce = flat[cell + 1];
        }
        const int cnt = ce - cs, incl = wave_scan(cnt);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        for (int f0 = 0; f0 < total; f0 += 64) {
          // the first subcell of the group whose prefix sum exceeds f
          const int f = f0 + lane;
          int g = 0;
#pragma unroll
          for (int o = 32; o > 0; o >>= 1)
            if (__shfl(incl, g + o - 1) <= f) g += o;
          const int q = __shfl(cs, g) + f - (__shfl(incl, g) - __shfl(cnt, g));
          if (f < total) {
            if (q == p) continue;
            double xq[D];
            load_x<D>(xb, q, xq);
            double r2 = 0.0;
            for (int a = 0; a < D; a++) {
              const double dx = min_image(xq[a] - xp[a], L, h);
              r2 = __builtin_fma(dx, dx, r2);
            }
            // no diameter reaches further (most of the linked subcells' atoms:
            // their diameters, each a load past the caches, are not read)
            if (!(r2 < far2)) continue;
            const double sq = sig_get(xb + (size_t)q * DR + D);
            double fc, uu;
            const double s_b = 0.5 * (sa + sq);
            if (r2 < (cut * s_b) * (cut * s_b)) {
              if (morse) pair_f64<true>(pot, eps, ma, r2, s_b, fc, uu);
              else pair_f64<false>(pot, eps, ma, r2, s_b, fc, uu);
              eb += uu;
            }
            // after the exchange the partner carries p's old diameter
            const double s_a = 0.5 * (sb + (q == o ? sa : sq));
            if (r2 < (cut * s_a) * (cut * s_a)) {
              if (morse) pair_f64<true>(pot, eps, ma, r2, s_a, fc, uu);
              else pair_f64<false>(pot, eps, ma, r2, s_a, fc, uu);
              ea += uu;
            }
          }
        }
      }
    }
  }
  eb = wave_sum(eb);
  ea = wave_sum(ea);
  if (lane == 0) {
    red[0][wv] = eb;
    red[1][wv] = ea;
  }
  __syncthreads();
  eb = 0.0;
  ea = 0.0;
  for (int w = 0; w < nwv; w++) {
    eb += red[0][w];
    ea += red[1][w];
  }
  __syncthreads();  // red[] is free again
  return pi == pj ? 0.0 : ea - eb;
}

// The batch of a round: the nput attempts put off by the previous round
// (off_in, in order) followed by the attempts cursor, cursor + 1, ... not yet
// begun; kSwapBatch of them at most.  ctl[0] = nput, ctl[2] = cursor.
__device__ inline int swap_batch_size(const long long* ctl, int64_t n_att) {
  const long long rest = (long long)n_att - ctl[2];
  const long long nb = ctl[0] + rest;
  return (int)(nb < kSwapBatch ? nb : kSwapBatch);
}
__device__ inline int swap_attempt(const long long* ctl, const int32_t* off_in, int b) {
  const int nput = (int)ctl[0];
  return b < nput ? off_in[b] : (int)(ctl[2] + (b - nput));
}

// dE of the round's attempts, one workgroup each, with the two diameters it
// was taken with: de[3b] = dE, de[3b+1], de[3b+2] = the diameters of the
// first and the second atom.  conf[b][w] bit c: attempt b' = 64 w + c < b
// has an atom within c sigma_max of an atom of attempt b.
template <int D>
__global__ __launch_bounds__(1024) void k_swap_de(const SysDev* s, const long long* __restrict__ ctl,
                                                  const int32_t* __restrict__ off_in, int64_t n_att,
                                                  const int32_t* __restrict__ pairs,
                                                  const int32_t* __restrict__ slot_of,
                                                  double* __restrict__ de,
                                                  unsigned long long* __restrict__ conf) {
  __shared__ double red[2][16];
  const int b = blockIdx.x;
  const int nb = swap_batch_size(ctl, n_att);
  if (b >= nb) return;
  const int k = swap_attempt(ctl, off_in, b);
  const int pi = slot_of[pairs[2 * k]], pj = slot_of[pairs[2 * k + 1]];
  {
    const double* xb = s->x[s->xcur];
    const double L = s->L, h = s->hL;
    const double rr = s->cutoff * s->sigma_max, r2max = rr * rr * (1.0 + 1e-12);
    const int t = threadIdx.x;
    bool near = false;
    if (t < b) {
      const int k2 = swap_attempt(ctl, off_in, t);
      const int q2[2] = {slot_of[pairs[2 * k2]], slot_of[pairs[2 * k2 + 1]]};
      for (int e = 0; e < 4; e++) {
        double xa[D], xc[D];
        load_x<D>(xb, (e >> 1) ? pj : pi, xa);
        load_x<D>(xb, q2[e & 1], xc);
        double r2 = 0.0;
        for (int a = 0; a < D; a++) {
          const double dx = min_image(xa[a] - xc[a], L, h);
          r2 += dx * dx;
        }
        near = near || r2 <= r2max;
      }
    }
    const unsigned long long m = __ballot(near);
    if (t < kSwapBatch && (t & 63) == 0) conf[(size_t)b * (kSwapBatch / 64) + (t >> 6)] = m;
  }
  double si, sj;
  const double d = swap_de<D>(s, pi, pj, red, si, sj);
  if (threadIdx.x == 0) {
    de[3 * b] = d;
    de[3 * b + 1] = si;
    de[3 * b + 2] = sj;
  }
}

// Settles the round's batch in order (see above), applies the kept exchanges,
// and writes the attempts put off to off_out; ctl[0] = their number, ctl[2]
// advances past the attempts begun, ctl[1] += exchanges kept.  Only the
// decisions hang together: one wave takes 64 attempts at a time, the
// conflicts with the groups before in parallel, those inside the group one
// after the other in scalar registers; the exchanges kept touch no atom in
// common and are applied by all threads (one thread walking the batch with
// the stores in its chain took 82 us for 256 attempts, this 21).
template <int D>
__global__ __launch_bounds__(kSwapBatch) void k_swap_settle(SysDev* s, long long* __restrict__ ctl,
                                                      const int32_t* __restrict__ off_in,
                                                      int32_t* __restrict__ off_out, int64_t n_att,
                                                      const int32_t* __restrict__ pairs,
                                                      const double* __restrict__ u, double T,
                                                      const int32_t* __restrict__ slot_of,
                                                      const double* __restrict__ de,
                                                      const unsigned long long* __restrict__ cfg,
                                                      int32_t* __restrict__ acc,
                                                      double* __restrict__ diam) {
  constexpr int DR = Dims<D>::DR, NW = kSwapBatch / 64;
  __shared__ unsigned long long put[NW], kept[NW];  // per attempt: put off; settled and kept
  const int tid = threadIdx.x, lane = tid & 63;
  const int nb = swap_batch_size(ctl, n_att);
  if (nb <= 0) return;
  const int nput = (int)ctl[0];
  double* xb = s->x[s->xcur];
  if (tid < 64) {
    unsigned long long blk[NW], hits[NW], oks[NW];
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const int b = 64 * w + lane;
      const bool in = b < nb;
      // the decision of an attempt that settles (its dE stands)
      bool ok = false;
      if (in) {
        const int k = swap_attempt(ctl, off_in, b);
        const double d = de[3 * b];
        ok = d <= 0.0 || u[k] < exp(-d / T);
      }
      const unsigned long long okm = __ballot(ok);
      bool before = false;
#pragma unroll
      for (int v = 0; v < NW; v++)
        if (v < w && in) before = before || (cfg[(size_t)b * NW + v] & blk[v]) != 0;
      const unsigned long long own = in ? cfg[(size_t)b * NW + w] : 0ull;
      const unsigned long long pre = __ballot(before);
      unsigned long long hit = 0ull, bl = 0ull;
      const int cnt = min(max(nb - 64 * w, 0), 64);
      for (int c = 0; c < cnt; c++) {
        const unsigned long long m =
            ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(own >> 32), c) << 32) |
            (unsigned)__builtin_amdgcn_readlane((int)(unsigned)own, c);
        const bool h = ((pre >> c) & 1ull) != 0 || (m & bl) != 0;
        if (h) hit |= 1ull << c;
        if (h || ((okm >> c) & 1ull)) bl |= 1ull << c;
      }
      blk[w] = bl;
      hits[w] = hit;
      oks[w] = okm & ~hit;
    }
#pragma unroll
    for (int w = 0; w < NW; w++) {
      if (lane == 0) {
        put[w] = hits[w];
        kept[w] = oks[w];
      }
    }
  }
  __syncthreads();
  int noff = 0, nkept = 0;
  for (int w = 0; w < NW; w++) {
    noff += __popcll(put[w]);
    nkept += __popcll(kept[w]);
  }
  // off_in and ctl are read before any thread writes ctl (off_out is another array)
  if (tid < nb) {
    const int b = tid, w = b >> 6, k = swap_attempt(ctl, off_in, b);
    if (put[w] >> (b & 63) & 1ull) {
      int at = __popcll(put[w] & ((1ull << (b & 63)) - 1));
      for (int v = 0; v < w; v++) at += __popcll(put[v]);
      off_out[at] = k;
    } else {
      const bool ok = kept[w] >> (b & 63) & 1ull;
      if (acc) acc[k] = ok ? 1 : 0;
      if (ok) {
        // a settled attempt's atoms were not touched earlier in the batch, so
        // their diameters are the ones its dE was taken with
        const int c0 = pairs[2 * k], c1 = pairs[2 * k + 1];
        const double si = de[3 * b + 1], sj = de[3 * b + 2];
        sig_put(xb + (size_t)slot_of[c0] * DR + D, sj);
        sig_put(xb + (size_t)slot_of[c1] * DR + D, si);
        diam[c0] = sj;
        diam[c1] = si;
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    ctl[2] += nb - nput;
    ctl[0] = noff;
    ctl[1] += nkept;
  }
}

// Own atom's data as the force loop needs it.
template <int D, bool MIX>
struct Own {
  double x[D];  // FP64 coordinates
  double sg;
  int u[D];     // fixed-point coordinates (mixed)
};

// Entries of row i that may interact at the current positions.
__device__ inline int row_reach(const SysDev* s, int i) {
  return s->nshell == 1 ? min(gbl(s->nlen)[i], s->width)
                        : (int)gbl(s->ends)[(size_t)i * kShells + s->shells - 1];
}

// Partial force of lane `sub` of the LPA lanes that share slot i: entries
// k = sub, sub + LPA, ...; the next group's row indices are fetched before
// the current group's records are used.  The LPA partial sums are combined
// with the same butterfly on every lane of the group.
template <int D, bool MIX, int LPA, typename FT, bool MORSE>
__device__ inline void force_part(const SysDev* s, int i, bool vi, int sub, const Own<D, MIX>& me,
                                  FT (&F)[D], double& e, double& w, double& z) {
  constexpr int U = MIX ? 4 : 2;
  const int npad = s->npad, jmask = s->jmask;
  const int len = vi ? row_reach(s, i) : 0;
  const HDMD_GLOBAL int* __restrict__ nl = gbl(s->nl);
  const double L = s->L, c = s->cutoff, eps = s->eps, invL = 1.0 / L, ma = s->morse_a;
  const int pot = s->potential;
  const double* __restrict__ xb = s->x[s->xcur];
  const int32_t* __restrict__ qb = MIX ? s->q[s->xcur] : nullptr;
  const double fxinv = s->fxinv;
  // forces are summed in FP64 in both forms (the precision form stores them
  // as FP32): summing ~10^2-10^3 terms of mixed sign in FP32 would lose more
  // than 1e-5 of F_rms at high overlap
  double Fs[D];
#pragma unroll
  for (int k = 0; k < D; k++) Fs[k] = 0.0;
  e = 0.0;
  w = 0.0;
  z = 0.0;
  // row entries are read unconditionally from a clamped (in-bounds) slot and
  // masked afterwards, so the loads issue without branches and the wait for
  // the current group does not also wait for the prefetched one
  const int wm1 = s->width - 1;
  int jn[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int kk = sub + u * LPA;
    const int raw = nl[(size_t)min(kk, wm1) * npad + i];
    jn[u] = kk < len ? raw & jmask : -1;
  }
  for (int k0 = sub; k0 < len; k0 += U * LPA) {
    int jj[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      jj[u] = jn[u];
      const int kk = k0 + (U + u) * LPA;
      const int raw = nl[(size_t)min(kk, wm1) * npad + i];
      jn[u] = kk < len ? raw & jmask : -1;
    }
    if (!MIX) {
      double xj[U][D], sj[U];
#pragma unroll
      for (int u = 0; u < U; u++) load_rec<D>(xb, jj[u] >= 0 ? jj[u] : i, xj[u], sj[u]);
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (jj[u] < 0) continue;
        const double sij = 0.5 * (me.sg + sj[u]);
        const double rc = c * sij;
        double dx[D];
        double r2 = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
          dx[k] = near_image(xj[u][k] - me.x[k], L, invL);
          r2 = __builtin_fma(dx[k], dx[k], r2);
        }
        if (r2 < rc * rc) {
          double fc, uu;
          pair_f64<MORSE>(pot, eps, ma, r2, sij, fc, uu);
#pragma unroll
          for (int k = 0; k < D; k++) Fs[k] -= fc * dx[k];
          e += 0.5 * uu;
          w += 0.5 * fc * r2;
          z += 1.0;
        }
      }
    } else {
      // mixed: exact integer displacements; distance, pair coefficient and
      // force sum in FP64 (stored as FP32 by the caller)
      int uj[U][D];
      double sj[U];
#pragma unroll
      for (int u = 0; u < U; u++) load_q<D>(qb, jj[u] >= 0 ? jj[u] : i, uj[u], sj[u]);
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (jj[u] < 0) continue;
        const double sij = 0.5 * (me.sg + sj[u]);
        const double rc = c * sij;
        double dx[D];
        double r2 = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
          dx[k] = (double)(int)(uj[u][k] - me.u[k]) * fxinv;  // two's complement = minimum image
          r2 = __builtin_fma(dx[k], dx[k], r2);
        }
        if (r2 < rc * rc) {
          double fc, uu;
          pair_f64<MORSE>(pot, eps, ma, r2, sij, fc, uu);
#pragma unroll
          for (int k = 0; k < D; k++) Fs[k] -= fc * dx[k];
          e += 0.5 * uu;
          w += 0.5 * fc * r2;
          z += 1.0;
        }
      }
    }
  }
#pragma unroll
  for (int o = 1; o < LPA; o <<= 1) {
#pragma unroll
    for (int k = 0; k < D; k++) Fs[k] += __shfl_xor(Fs[k], o, 64);
    e += __shfl_xor(e, o, 64);
    w += __shfl_xor(w, o, 64);
    z += __shfl_xor(z, o, 64);
  }
#pragma unroll
  for (int k = 0; k < D; k++) F[k] = FT(Fs[k]);
}

// Partial force of one lane per atom (the whole row), with the neighbour
// records staged through LDS.  A gather in which every lane loads its own
// neighbour's record touches as many cache lines per load instruction as
// there are lanes; here the wave loads the records of R row entries of all 64
// lanes cooperatively (RB/16 lanes share one record, one 16-byte piece each,
// so an instruction covers 16 / 32 / 64 whole records) straight into LDS
// (global_load_lds_dwordx4), then every lane reads its own records back.  The
// pairs are summed in row order, exactly as force_part does, so the results
// are the same bits.  The loop runs to the longest row of the wave; the
// pieces of record r sit rotated by r in its LDS slot so that the lanes'
// reads spread over the banks.  stage: kStage16 16-byte slots of LDS.
constexpr int kStage16 = 512;  // 8 KiB per wave

template <int D, bool MIX>
struct StageGeom {
  static constexpr int RB = MIX ? Dims<D>::DQ * 4 : Dims<D>::DR * 8;  // record bytes
  static constexpr int PR = RB / 16;                                  // pieces per record
  static constexpr int R = kStage16 / (64 * PR);                      // rows entries per pass
};

template <int D, bool MIX, typename FT, bool MORSE>
__device__ inline void force_part_lds(const SysDev* s, int i, bool vi, const Own<D, MIX>& me,
                                      FT (&F)[D], double& e, double& w, double& z, vd2* stage) {
  typedef StageGeom<D, MIX> G;
  constexpr int PR = G::PR, R = G::R, RPI = 64 / PR;  // records per load instruction
  static_assert(R >= 1 && R * 64 * PR <= kStage16, "stage size");
  const int lane = threadIdx.x & 63;
  const int npad = s->npad, W = s->width, jmask = s->jmask;
  const int len = vi ? row_reach(s, i) : 0;
  const int mx = uniform_int(wave_max_i(len));
  const HDMD_GLOBAL int* __restrict__ nl = gbl(s->nl);
  const double L = s->L, c = s->cutoff, eps = s->eps, invL = 1.0 / L, ma = s->morse_a;
  const int pot = s->potential;
  const char* __restrict__ base =
      MIX ? reinterpret_cast<const char*>(s->q[s->xcur]) : reinterpret_cast<const char*>(s->x[s->xcur]);
  const double fxinv = s->fxinv;
  double Fs[D];
#pragma unroll
  for (int k = 0; k < D; k++) Fs[k] = 0.0;
  e = 0.0;
  w = 0.0;
  z = 0.0;
  for (int k0 = 0; k0 < mx; k0 += R) {
    int j[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
      const int kk = k0 + r;
      const int raw = nl[(size_t)min(kk, W - 1) * npad + i];
      j[r] = kk < len ? raw & jmask : -1;
    }
    wave_lds_sync();  // the previous pass's reads of the stage are done
#pragma unroll
    for (int r = 0; r < R; r++) {
#pragma unroll
      for (int q = 0; q < PR; q++) {
        // lane t loads piece ((t % PR) - rec) mod PR of record rec = q RPI + t / PR
        // of this round into slot t % PR: LDS byte 16 t of the instruction's 1 KiB
        const int rec = q * RPI + lane / PR;
        const int jr = PR == 1 ? j[r] : __shfl(j[r], rec, 64);
        const int piece = ((lane % PR) - rec) & (PR - 1);
        const char* src = base + (size_t)(jr >= 0 ? jr : 0) * G::RB + 16 * piece;
        __builtin_amdgcn_global_load_lds((const void*)src, (void*)(stage + (r * PR + q) * 64), 16, 0,
                                         0);
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < R; r++) {
      // own record of this round: pieces p at slots (p + lane) mod PR
      const vd2* rec = stage + r * PR * 64 + lane * PR;
      if (!MIX) {
        double xj[D], sj = 0.0;
        vd2 pc[PR];
#pragma unroll
        for (int p = 0; p < PR; p++) pc[p] = rec[(p + lane) & (PR - 1)];
#pragma unroll
        for (int k = 0; k < D; k++) xj[k] = (k & 1) ? pc[k >> 1].y : pc[k >> 1].x;
        sj = (D & 1) ? pc[D >> 1].y : pc[D >> 1].x;
        if (j[r] < 0) continue;
        const double sij = 0.5 * (me.sg + sj);
        const double rc = c * sij;
        double dx[D];
        double r2 = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
          dx[k] = near_image(xj[k] - me.x[k], L, invL);
          r2 = __builtin_fma(dx[k], dx[k], r2);
        }
        if (r2 < rc * rc) {
          double fc, uu;
          pair_f64<MORSE>(pot, eps, ma, r2, sij, fc, uu);
#pragma unroll
          for (int k = 0; k < D; k++) Fs[k] -= fc * dx[k];
          e += 0.5 * uu;
          w += 0.5 * fc * r2;
          z += 1.0;
        }
      } else {
        constexpr int SQ = Dims<D>::SQ;
        int v[4 * PR];
#pragma unroll
        for (int p = 0; p < PR; p++) {
          const vi4 t = reinterpret_cast<const vi4*>(rec)[(p + lane) & (PR - 1)];
          v[4 * p] = t.x;
          v[4 * p + 1] = t.y;
          v[4 * p + 2] = t.z;
          v[4 * p + 3] = t.w;
        }
        const double sj = __longlong_as_double(
            (long long)(((unsigned long long)(unsigned)v[SQ + 1] << 32) | (unsigned)v[SQ]));
        if (j[r] < 0) continue;
        const double sij = 0.5 * (me.sg + sj);
        const double rc = c * sij;
        double dx[D];
        double r2 = 0.0;
#pragma unroll
        for (int k = 0; k < D; k++) {
          dx[k] = (double)(int)(v[k] - me.u[k]) * fxinv;  // two's complement = minimum image
          r2 = __builtin_fma(dx[k], dx[k], r2);
        }
        if (r2 < rc * rc) {
          double fc, uu;
          pair_f64<MORSE>(pot, eps, ma, r2, sij, fc, uu);
#pragma unroll
          for (int k = 0; k < D; k++) Fs[k] -= fc * dx[k];
          e += 0.5 * uu;
          w += 0.5 * fc * r2;
          z += 1.0;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < D; k++) F[k] = FT(Fs[k]);
}

template <int D, bool MIX>
__device__ inline void load_own(const SysDev* s, int i, Own<D, MIX>& me) {
  load_rec<D>(s->x[s->xcur], i, me.x, me.sg);
  if (MIX) {
    double sgq;
    load_q<D>(s->q[s->xcur], i, me.u, sgq);
  }
}

template <bool MIX>
struct VType {
  typedef double T;
};
template <>
struct VType<true> {
  typedef float T;
};

// Per-tile partial sums of the slots in `use` (a bit per Part; the others
// are left as they are and read by nobody): each wave reduces its lanes, then
// (LPA > 1) thread 0 adds the waves of the tile in order (deterministic for a
// given LPA).  `use` is uniform over the block.
constexpr unsigned kUseForce = (1u << P_PE) | (1u << P_FV) | (1u << P_FF) | (1u << P_VV) |
                               (1u << P_FMAX2);
constexpr unsigned kUseStep = (1u << P_PE) | (1u << P_KE) | (1u << P_FMAX2) | (1u << P_VIR) |
                              (1u << P_NC);
constexpr unsigned kUseDisp = (1u << P_M2) | (1u << P_M4) | (1u << P_OV);

template <int LPA>
__device__ inline void tile_partials(double* dst, double (&vals)[kPart], double& maxv,
                                     double* sh, unsigned use) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int p = 0; p < kPart; p++)
    if (p != P_FMAX2 && (use >> p & 1u)) vals[p] = wave_sum(vals[p]);
  maxv = wave_max(maxv);
  if (LPA == 1) {
    if (lane == 0) {
#pragma unroll
      for (int p = 0; p < kPart; p++)
        if (use >> p & 1u) dst[p] = p == P_FMAX2 ? maxv : vals[p];
    }
    return;
  }
  if (lane == 0) {
#pragma unroll
    for (int p = 0; p < kPart; p++)
      if (use >> p & 1u) sh[w * kPart + p] = p == P_FMAX2 ? maxv : vals[p];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int p = 0; p < kPart; p++) {
      if (!(use >> p & 1u)) continue;
      double acc = sh[p];
      for (int ww = 1; ww < LPA; ww++)
        acc = p == P_FMAX2 ? fmax(acc, sh[ww * kPart + p]) : acc + sh[ww * kPart + p];
      dst[p] = acc;
    }
  }
  __syncthreads();
}

// One atom tile's forces (stored in s->f) with the tile's energy and, for
// FIRE, the power P = F.v, |F|^2, |v|^2 and max_i |F_i|^2 partial sums.
// The force kernels serve the systems of one potential class: MORSE, or WCA
// and harmonic (run-time switch); of one precision form; and of one number
// of lanes per atom.
__device__ inline bool kernel_serves(const SysDev* s, bool mix, bool morse, int lpa) {
  return (s->precision != 0) == mix && (s->potential == kPotMorse) == morse && s->lpa == lpa;
}

template <int D, bool MIX, int LPA, bool MORSE>
__device__ inline void force_tile(SysDev* s, int tile, int fire, double* sh, vd2* stage) {
  typedef typename VType<MIX>::T FT;
  const int sub = threadIdx.x % LPA, slot = threadIdx.x / LPA;
  const int i = tile * kTile + slot;
  const int n = s->n, npad = s->npad, pc = s->pcur;
  const bool vi = i < n;
  const int ii = vi ? i : 0;
  Own<D, MIX> me;
  load_own<D, MIX>(s, ii, me);
  FT F[D];
  double e, w, z;
  if constexpr (LPA == 1) force_part_lds<D, MIX, FT, MORSE>(s, ii, vi, me, F, e, w, z, stage);
  else force_part<D, MIX, LPA, FT, MORSE>(s, ii, vi, sub, me, F, e, w, z);
  double vals[kPart], mx = 0.0;
#pragma unroll
  for (int p = 0; p < kPart; p++) vals[p] = 0.0;
  if (vi && sub == 0) {
    FT* fo = reinterpret_cast<FT*>(s->f);
    const FT* v = reinterpret_cast<const FT*>(s->v[pc]);
    double fv = 0.0, ff = 0.0, vv = 0.0;
#pragma unroll
    for (int k = 0; k < D; k++) {
      fo[(size_t)k * npad + i] = F[k];
      if (fire) {
        const double fk = (double)F[k], vk = (double)v[(size_t)k * npad + i];
        fv += fk * vk;
        ff += fk * fk;
        vv += vk * vk;
      }
    }
    vals[P_PE] = e;
    vals[P_FV] = fv;
    vals[P_FF] = ff;
    vals[P_VV] = vv;
    mx = ff;
  }
  tile_partials<LPA>(s->part + (size_t)tile * kPart, vals, mx, sh, kUseForce);
}

template <int D, bool MIX, int LPA, bool MORSE>
__global__ __launch_bounds__(kTile * LPA) void k_force(KArgs a, int fire) {
  __shared__ double sh[LPA * kPart];
  __shared__ vd2 stage[LPA == 1 ? kStage16 : 1];
  for (int t = xcd_tile(blockIdx.x, gridDim.x);; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile(a, t, s, tile)) break;
    if (!live(s) || !kernel_serves(s, MIX, MORSE, LPA)) continue;
    if (fire && s->mode != MODE_FIRE) continue;
    force_tile<D, MIX, LPA, MORSE>(s, tile, fire, sh, stage);
  }
}

// Fused velocity-Verlet step (kick-drift-kick leapfrog, Sec. II.B):
//   F = F(x^n); v^n = lambda (v^(n-1/2) + dt/2 F) (skipped at step 0, where v
//   is the full-step velocity; lambda is the Berendsen factor from the
//   previous full step's temperature, 1 without a thermostat: the paper folds
//   the thermostat into this kick); record KE(v^n), PE(x^n); v^(n+1/2) = v^n + dt/2 F;
//   x^(n+1) = wrap(x^n + dt v^(n+1/2)) into the other record buffer;
//   max_i |x^(n+1)_i - x_ref,i|^2 for the rebuild trigger (skin/2).
// At the closing step (n == nsteps) only the second kick is applied.
// On steps that record a thermo row, the unwrapped displacement since the
// run's start, Delta_i = disp_i + (x^n_i - x_ref,i), gives |Delta|^2,
// |Delta|^4 and the overlap term Theta(0.1 d - |Delta|) (Sec. II.E, eqs. ngp
// and fov); disp_i is advanced at each rebuild, so other steps read nothing.
template <int D, bool MIX, int LPA, bool MORSE>
__global__ __launch_bounds__(kTile * LPA) void k_step(KArgs a) {
  typedef typename VType<MIX>::T VT;
  __shared__ double sh[LPA * kPart];
  __shared__ vd2 stage[LPA == 1 ? kStage16 : 1];
  const int sub = threadIdx.x % LPA, slot = threadIdx.x / LPA;
  for (int t = xcd_tile(blockIdx.x, gridDim.x);; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile(a, t, s, tile)) break;
    if (!live(s) || s->mode != MODE_MD || !kernel_serves(s, MIX, MORSE, LPA)) continue;
    const int i = tile * kTile + slot;
    const int n = s->n, npad = s->npad, pc = s->pcur, cur = s->xcur;
    const bool vi = i < n;
    const int ii = vi ? i : 0;
    const bool first = s->step == 0, close = s->step >= s->nsteps;
    const bool rec = s->thermo && s->thermo_every > 0 && s->step % s->thermo_every == 0;
    const double dt = s->dt, hdt = 0.5 * dt;
    Own<D, MIX> me;
    load_own<D, MIX>(s, ii, me);
    VT F[D];
    double e, w, z;
    if constexpr (LPA == 1) force_part_lds<D, MIX, VT, MORSE>(s, ii, vi, me, F, e, w, z, stage);
    else force_part<D, MIX, LPA, VT, MORSE>(s, ii, vi, sub, me, F, e, w, z);
    double vals[kPart], mx = 0.0;
#pragma unroll
    for (int p = 0; p < kPart; p++) vals[p] = 0.0;
    if (vi && sub == 0) {
      VT* v = reinterpret_cast<VT*>(s->v[pc]);
      const VT lam = VT(s->vscale);
      const double L = s->L, h = s->hL;
      double m2 = 0.0;
      if (rec) {
#pragma unroll
        for (int k = 0; k < D; k++) {
          const size_t o = (size_t)k * npad + i;
          const double dd = s->disp[pc][o] + min_image(me.x[k] - s->xref[o], L, h);
          m2 = __builtin_fma(dd, dd, m2);
        }
      }
      VT vk[D];
      double xn[D], ke = 0.0;
#pragma unroll
      for (int k = 0; k < D; k++) {
        vk[k] = v[(size_t)k * npad + i];
        if (!first) vk[k] = lam * (vk[k] + VT(hdt) * F[k]);
        ke += (double)vk[k] * (double)vk[k];
      }
      double r2 = 0.0;
#pragma unroll
      for (int k = 0; k < D; k++) {
        if (!close) {
          vk[k] += VT(hdt) * F[k];
          xn[k] = wrap1(me.x[k] + dt * (double)vk[k], L, h);
        } else {
          xn[k] = me.x[k];
        }
        v[(size_t)k * npad + i] = vk[k];
        const double dx = min_image(xn[k] - s->xref[(size_t)k * npad + i], L, h);
        r2 = __builtin_fma(dx, dx, r2);
      }
      store_rec<D>(s->x[cur ^ 1], i, xn, me.sg);
      if (MIX) store_q<D>(s->q[cur ^ 1], i, xn, me.sg, h, s->fxscale);
      vals[P_PE] = e;
      vals[P_KE] = 0.5 * ke;
      vals[P_VIR] = w;
      vals[P_NC] = z;
      vals[P_M2] = m2;
      vals[P_M4] = m2 * m2;
      vals[P_OV] = rec && m2 < 0.01 * D * D ? 1.0 : 0.0;
      mx = r2;
    }
    // the displacement maximum of the tile is reduced like the partial sums
    double* pt = s->part + (size_t)tile * kPart;
    tile_partials<LPA>(pt, vals, mx, sh, kUseStep | kUseDisp);
    if (threadIdx.x == 0 && pt[P_FMAX2] > 0.0)
      atomicMax(&s->maxdisp2, (unsigned long long)__double_as_longlong(pt[P_FMAX2]));
  }
}

// FIRE 2.0 semi-implicit Euler update with the coefficients of this
// iteration (computed per system by fire_control):
//   on P <= 0: x -= dt/2 v, v = 0;  v += dt F;  v = (1-a) v + a |v|/|F| F;
//   x += dt v (wrapped, into the other buffer); displacement for the trigger.
template <int D, bool MIX>
__device__ inline void fire_update_tile(SysDev* s, int tile, double dt, double keep, double mix,
                                        bool zero) {
  typedef typename VType<MIX>::T VT;
  const int i = tile * kTile + threadIdx.x;
  const int n = s->n, npad = s->npad, pc = s->pcur, cur = s->xcur;
  double disp2 = 0.0;
  if (i < n) {
    const double L = s->L, h = s->hL;
    double x[D], sg;
    load_rec<D>(s->x[cur], i, x, sg);
    VT* v = reinterpret_cast<VT*>(s->v[pc]);
    const VT* f = reinterpret_cast<const VT*>(s->f);
    double r2 = 0.0;
#pragma unroll
    for (int k = 0; k < D; k++) {
      double vk = (double)v[(size_t)k * npad + i];
      const double fk = (double)f[(size_t)k * npad + i];
      if (zero) {
        x[k] = x[k] - 0.5 * dt * vk;
        vk = 0.0;
      }
      vk = vk + dt * fk;
      vk = keep * vk + mix * fk;
      const VT vs = VT(vk);
      v[(size_t)k * npad + i] = vs;
      x[k] = wrap1(x[k] + dt * (double)vs, L, h);
      double dx = min_image(x[k] - s->xref[(size_t)k * npad + i], L, h);
      r2 = __builtin_fma(dx, dx, r2);
    }
    store_rec<D>(s->x[cur ^ 1], i, x, sg);
    if (MIX) store_q<D>(s->q[cur ^ 1], i, x, sg, h, s->fxscale);
    disp2 = r2;
  }
  const double dm = wave_max(disp2);
  if ((threadIdx.x & (kWave - 1)) == 0 && dm > 0.0)
    atomicMax(&s->maxdisp2, (unsigned long long)__double_as_longlong(dm));
}

// One system alone.  Up to kFireFused tiles every workgroup takes the
// control's decision itself (the same bits in each), and the finalisation
// writes it to the descriptor, which no workgroup reads then.
template <int D, bool MIX>
__global__ __launch_bounds__(kTile) void k_fire_update(KArgs a) {
  SysDev* s = a.single;
  const int tile = blockIdx.x;
  if (!live(s) || s->mode != MODE_FIRE || tile >= s->ntiles) return;
  if (a.fin == 2) {
    const FireNext f = fire_control(s);
    if (tile == 0 && threadIdx.x == 0) s->fnext = f;
    if (f.status == SLOT_RUNNING)
      fire_update_tile<D, MIX>(s, tile, f.fdt, f.c_keep, f.c_mix, f.zero != 0);
  } else {
    fire_update_tile<D, MIX>(s, tile, s->fdt, s->c_keep, s->c_mix, s->c_zero != 0);
  }
}

}  // namespace hdmd

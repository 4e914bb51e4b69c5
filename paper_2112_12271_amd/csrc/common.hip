// common.hip -- dimension-independent kernels: descriptor upload, prefix
// sums of the subcell occupancies, counting-sort placement, per-system
// finalisation of a step (reductions, thermo rows, buffer flips) and the
// per-system FIRE 2.0 control.
#include "kernels.h"
#include "dispatch.h"

namespace hdmd {

const DKernels* dkernels_d2();
const DKernels* dkernels_d3();
const DKernels* dkernels_d4();
const DKernels* dkernels_d5();
const DKernels* dkernels_d6();
const DKernels* dkernels_d7();
const DKernels* dkernels_d8();
const DKernels* dkernels_d9();
const DKernels* dkernels_d10();

const DKernels* dkernels(int d) {
  switch (d) {
    case 2: return dkernels_d2();
    case 3: return dkernels_d3();
    case 4: return dkernels_d4();
    case 5: return dkernels_d5();
    case 6: return dkernels_d6();
    case 7: return dkernels_d7();
    case 8: return dkernels_d8();
    case 9: return dkernels_d9();
    case 10: return dkernels_d10();
    default: return nullptr;
  }
}

__global__ void k_setdesc(SysDev* dst, SysDev val) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = val;
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Snapshot of every slot's state and iteration / step count.
__global__ void k_poll(const Table* t, int32_t* state, int64_t* iters) {
  int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= t->max_slots) return;
  const SysDev* s = t->sys[slot];
  if (!s) {
    state[slot] = SLOT_EMPTY;
    iters[slot] = 0;
    return;
  }
  state[slot] = s->status;
  iters[slot] = s->mode == MODE_MD ? (s->step > 0 ? s->step - 1 : 0) : s->iters;
}

// Exclusive scan of the occupancies of one chunk of kChunk subcells.
__global__ __launch_bounds__(256) void k_scan1(KArgs a) {
  __shared__ int sh[256];
  const int tid = threadIdx.x;
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    int ch;
    if (!fetch_chunk_tile(a, t, s, ch)) break;
    if (!rebuilding(a, s)) {
      if (a.single) break;  // one system: the same for every tile
      continue;
    }
    const int nc = s->ncells;
    const int c0 = ch * kChunk + tid * 4;
    int v[4], local = 0;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      v[u] = (c0 + u < nc) ? s->cell_count[c0 + u] : 0;
      local += v[u];
    }
    sh[tid] = local;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
      int x = tid >= off ? sh[tid - off] : 0;
      __syncthreads();
      sh[tid] += x;
      __syncthreads();
    }
    int run = sh[tid] - local;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      if (c0 + u < nc) s->cell_local[c0 + u] = run;
      run += v[u];
    }
    if (tid == 255) s->chunk_sum[ch] = sh[255];
    __syncthreads();
  }
}

// Exclusive scan of the chunk totals of one system.
__global__ __launch_bounds__(256) void k_scan2(KArgs a) {
  __shared__ int sh[256];
  const int tid = threadIdx.x;
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    if (!fetch_sys(a, t, s)) break;
    if (!rebuilding(a, s)) {
      if (a.single) break;  // one system: the same for every tile
      continue;
    }
    int carry = 0;
    for (int b = 0; b < s->nchunks; b += 256) {
      const int c = b + tid;
      const int v = c < s->nchunks ? s->chunk_sum[c] : 0;
      sh[tid] = v;
      __syncthreads();
      for (int off = 1; off < 256; off <<= 1) {
        int x = tid >= off ? sh[tid - off] : 0;
        __syncthreads();
        sh[tid] += x;
        __syncthreads();
      }
      if (c < s->nchunks) s->chunk_off[c] = carry + sh[tid] - v;
      carry += sh[255];
      __syncthreads();
    }
    if (tid == 0) s->max_row = 0;
    __syncthreads();
  }
}

// Counting-sort placement: slot = start(subcell) + arrival rank.
__global__ __launch_bounds__(kTile) void k_scatter(KArgs a) {
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    int tile;
    if (!fetch_atom_tile(a, t, s, tile)) break;
    if (!rebuilding(a, s)) {
      if (a.single) break;  // one system: the same for every tile
      continue;
    }
    const int i = tile * kTile + threadIdx.x;
    if (i >= s->n) continue;
    scatter_atom(s, i, s->cell_of[i], s->rank[i]);
  }
}

// Finalisation of the systems of a batch (and of a system's first build).
__global__ __launch_bounds__(64) void k_finalize(KArgs a) {
  if (a.tab && blockIdx.x == 0 && threadIdx.x == 0) a.tab->build_waves = 0;
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    if (!fetch_sys(a, t, s)) break;
    finalize_system(s, need_rebuild(s));
  }
}

// FIRE 2.0 control of the systems of a batch and of large systems.
__global__ __launch_bounds__(64) void k_fire_ctrl(KArgs a) {
  for (int t = blockIdx.x;; t += gridDim.x) {
    SysDev* s;
    if (!fetch_sys(a, t, s)) break;
    if (!live(s) || s->mode != MODE_FIRE) continue;
    const FireNext f = fire_control(s);
    if (threadIdx.x == 0) fire_commit(s, f);
  }
}

// ---------------------------------------------------------------------------
// canonical CSR export (caller ids, ascending rows)
// ---------------------------------------------------------------------------
__global__ void k_export_lens(const SysDev* s, int64_t* row_ptr) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= s->n) return;
  row_ptr[s->oid[s->pcur][p] + 1] = min(s->nlen[p], s->width);
}

// All-ascending bitonic network; entries at index >= cnt act as +infinity, so
// any length works.
__device__ inline void bitonic_sort(int* keys, int cnt) {
  int p2 = 1;
  while (p2 < cnt) p2 <<= 1;
  const int half = p2 >> 1;
  auto cas = [&](int i, int p) {
    if (p < cnt && keys[i] > keys[p]) {
      const int k = keys[i];
      keys[i] = keys[p];
      keys[p] = k;
    }
  };
  for (int size = 2; size <= p2; size <<= 1) {
    const int hs = size >> 1;
    for (int t = threadIdx.x; t < half; t += blockDim.x) {
      const int blk = t / hs, off = t % hs;
      cas(blk * size + off, blk * size + size - 1 - off);
    }
    __syncthreads();
    for (int st = size >> 2; st > 0; st >>= 1) {
      for (int t = threadIdx.x; t < half; t += blockDim.x) {
        const int blk = t / st, off = t % st;
        const int i = blk * 2 * st + off;
        cas(i, i + st);
      }
      __syncthreads();
    }
  }
}

// Rows up to kRankRow entries: an entry's place is the number of smaller ones
// (all distinct), counted four to an LDS read; a bitonic network's chain of
// barriers took 182 us for 40009 rows of 150.  The count grows with the square
// of the row; longer rows keep the network.
constexpr int kRankRow = 512;

__global__ __launch_bounds__(256) void k_export_fill(const SysDev* s, const int64_t* row_ptr, int32_t* cols) {
  __shared__ __align__(16) int keys[kSortCap];
  const int p = blockIdx.x;
  if (p >= s->n) return;
  const int pc = s->pcur, npad = s->npad;
  const int a = s->oid[pc][p];
  const int len = min(s->nlen[p], s->width);
  int* out = cols + row_ptr[a];
  int* buf = len <= kSortCap ? keys : out;
  for (int k = threadIdx.x; k < len; k += blockDim.x) buf[k] = s->oid[pc][s->nl[(size_t)k * npad + p] & s->jmask];
  if (len <= kRankRow && (int)threadIdx.x < 4) keys[len + threadIdx.x] = INT32_MAX;
  __syncthreads();
  if (len <= kRankRow) {
    for (int k = threadIdx.x; k < len; k += blockDim.x) {
      const int me = keys[k];
      int r = 0;
      for (int q = 0; q < len; q += 4) {
        const int4 v = *reinterpret_cast<const int4*>(keys + q);
        r += (v.x < me) + (v.y < me) + (v.z < me) + (v.w < me);
      }
      out[r] = me;
    }
    return;
  }
  bitonic_sort(buf, len);
  if (buf == keys)
    for (int k = threadIdx.x; k < len; k += blockDim.x) out[k] = keys[k];
}

__global__ __launch_bounds__(256) void k_reduce_pe(const SysDev* s, double* out) {
  __shared__ double sh[256];
  const int tid = threadIdx.x;
  const int nw = s->nwaves, per = (nw + 255) / 256;
  double pe = 0.0;
  for (int w = tid * per; w < min(nw, (tid + 1) * per); w++) pe += s->part[(size_t)w * kPart + P_PE];
  pe = block_sum<256>(pe, sh);
  if (tid == 0) *out = pe;
}

// Inclusive scan of row lengths into CSR row pointers (row_ptr[0] = 0), by one
// workgroup, 8 rows per thread and pass: eight independent wave scans and one
// exchange, where a scan of 1024 rows at a time in LDS was a chain of twenty
// barriers (40009 rows: 79 us).
__global__ __launch_bounds__(1024) void k_export_scan(int n, int64_t* row_ptr) {
  constexpr int PER = 8, W = 16;
  __shared__ int64_t sh[W];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int64_t carry = 0;
  if (tid == 0) row_ptr[0] = 0;
  for (int64_t b = 0; b < n; b += 1024 * PER) {
    const int64_t c0 = b + w * 64 * PER + lane;
    int64_t x[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) x[u] = c0 + 64 * u < n ? row_ptr[c0 + 64 * u + 1] : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
      for (int u = 0; u < PER; u++) {
        const int64_t y = __shfl_up(x[u], o);
        if (lane >= o) x[u] += y;
      }
    }
    int64_t tot = 0;
#pragma unroll
    for (int u = 0; u < PER; u++) {
      const int64_t t = __shfl(x[u], 63);
      x[u] += tot;
      tot += t;
    }
    if (lane == 0) sh[w] = tot;
    __syncthreads();
    int64_t rest = 0;
    for (int q = 0; q < W; q++) {
      if (q < w) carry += sh[q];
      else rest += sh[q];
    }
#pragma unroll
    for (int u = 0; u < PER; u++)
      if (c0 + 64 * u < n) row_ptr[c0 + 64 * u + 1] = carry + x[u];
    carry += rest;
    __syncthreads();
  }
}

void launch_setdesc(SysDev* dst, const SysDev& val, hipStream_t st) {
  k_setdesc<<<1, 64, 0, st>>>(dst, val);
}
void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  if (n <= 0) return;
  int64_t g = (n + 255) / 256;
  k_fill_i32<<<(int)(g < 4096 ? g : 4096), 256, 0, st>>>(p, n, v);
}
void launch_scan1(const KArgs& a, int grid, hipStream_t st) { k_scan1<<<grid, 256, 0, st>>>(a); }
void launch_scan2(const KArgs& a, int grid, hipStream_t st) { k_scan2<<<grid, 256, 0, st>>>(a); }
void launch_scatter(const KArgs& a, int grid, hipStream_t st) {
  k_scatter<<<grid, kTile, 0, st>>>(a);
}
void launch_finalize(const KArgs& a, int grid, hipStream_t st) {
  k_finalize<<<grid, 64, 0, st>>>(a);
}
void launch_fire_ctrl(const KArgs& a, int grid, hipStream_t st) {
  k_fire_ctrl<<<grid, 64, 0, st>>>(a);
}
// slot_of[caller id] = position in subcell order
__global__ __launch_bounds__(256) void k_slot_of(const SysDev* s, int32_t* slot_of) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p < s->n) slot_of[s->oid[s->pcur][p]] = p;
}

void launch_slot_of(const SysDev* s, int n, int32_t* slot_of, hipStream_t st) {
  k_slot_of<<<(n + 255) / 256, 256, 0, st>>>(s, slot_of);
}

// SWAP set-up: zeroes the round counters (ctl[0..2]) and flags in ctl[3] any
// pair id outside [0, n).
__global__ __launch_bounds__(256) void k_swap_init(int64_t n_att, const int32_t* pairs, int n,
                                                   long long* ctl) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t == 0) {
    ctl[0] = 0;
    ctl[1] = 0;
    ctl[2] = 0;
  }
  bool bad = false;
  for (int64_t k = t; k < 2 * n_att; k += (int64_t)gridDim.x * 256) {
    const int32_t v = pairs[k];
    bad = bad || v < 0 || v >= n;
  }
  if (bad) atomicOr(reinterpret_cast<unsigned long long*>(ctl + 3), 1ull);
}

void launch_swap_init(int64_t n_att, const int32_t* pairs, int n, long long* ctl, hipStream_t st) {
  const int64_t g = (2 * n_att + 255) / 256;
  k_swap_init<<<(int)(g < 1 ? 1 : (g > 1024 ? 1024 : g)), 256, 0, st>>>(n_att, pairs, n, ctl);
}

void launch_reduce_pe(const SysDev* s, double* out, hipStream_t st) {
  k_reduce_pe<<<1, 256, 0, st>>>(s, out);
}
void launch_export(const SysDev* s, int n, int64_t* row_ptr, int32_t* cols, hipStream_t st,
                   int phase) {
  if (phase == 0) k_export_lens<<<(n + 255) / 256, 256, 0, st>>>(s, row_ptr);
  else if (phase == 1) k_export_scan<<<1, 1024, 0, st>>>(n, row_ptr);
  else k_export_fill<<<n, 256, 0, st>>>(s, row_ptr, cols);
}
void launch_poll(const Table* t, int max_slots, int32_t* state, int64_t* iters, hipStream_t st) {
  k_poll<<<(max_slots + 255) / 256, 256, 0, st>>>(t, state, iters);
}

}  // namespace hdmd

// nem_sort.hip -- binning of particles into cells (counting sort), ingest of
// host states, export to id order, and the per-step bookkeeping kernels.
//
// Particles are kept sorted by (replica, cell, id): every cell is a contiguous
// run and the order inside a cell is canonical, so results do not depend on
// the order in which atomics land. Rebinning happens only when some particle
// has left its cell by more than skin/2 (pass D raises a request); the two
// rebin kernels read it themselves and return at once when it is clear, so the
// per-step launch sequence is fixed.
#include "nem_dev.h"
#include "nem_pair.h"

namespace nem {



__device__ inline int rep_of_particle(const RepDev* reps, int R, int k) {
  int lo = 0, hi = R;  // largest r with part_base <= k
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (reps[mid].part_base <= k) lo = mid; else hi = mid;
  }
  return lo;
}

// Host state (FP64, id order) of replica r -> unsorted staging arrays.
// Takes the first predictor half-step in double precision:
// u^{n+1/2} = u^n + a dt/2, r^{n+1/2} = wrap(r^n + u^{n+1/2} dt/2).
__global__ void k_ingest(SortArgs s, int r, const double* __restrict__ in, int n, unsigned* umax) {
  const RepDev R = s.reps[r];
  const double* x = in;
  const double* y = in + n;
  const double* ux = in + 2 * (size_t)n;
  const double* uy = in + 3 * (size_t)n;
  const double* qxx = in + 4 * (size_t)n;
  const double* qxy = in + 5 * (size_t)n;
  const double* rho = in + 6 * (size_t)n;
  const double* ax = in + 7 * (size_t)n;
  const double* ay = in + 8 * (size_t)n;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
#pragma clang fp contract(off)
    const double hdt = 0.5 * (double)R.dt;
    const double uhx = ux[i] + hdt * ax[i], uhy = uy[i] + hdt * ay[i];
    double xh = x[i] + hdt * uhx, yh = y[i] + hdt * uhy;
    // wrap into [0, L), counting the periodic images taken off
    double ix = floor(xh / R.Ld), iy = floor(yh / R.Ld);
    xh = xh - R.Ld * ix; if (xh >= R.Ld) { xh -= R.Ld; ix += 1.0; } if (xh < 0.0) xh = 0.0;
    yh = yh - R.Ld * iy; if (yh >= R.Ld) { yh -= R.Ld; iy += 1.0; } if (yh < 0.0) yh = 0.0;
    if (!(fabs(ix) < 1e9 && fabs(iy) < 1e9)) { atomicOr(s.flags, ERR_RANGE); ix = 0.0; iy = 0.0; }
    int cx = (int)floor(xh / R.csd), cy = (int)floor(yh / R.csd);
    cx = min(max(cx, 0), R.nc - 1);
    cy = min(max(cy, 0), R.nc - 1);
    const double bx = (double)cx * R.csd, by = (double)cy * R.csd;
    const double ox = xh - bx, oy = yh - by;
    const float hx = (float)ox, hy = (float)oy;
    const float lx = (float)(ox - (double)hx), ly = (float)(oy - (double)hy);
    const int k = R.part_base + i;
    const int key = R.cell_base + cy * R.nc + cx;
    s.t_key[k] = key;
    s.t_off[k] = make_float2(hx, hy);
    s.t_lo[k] = make_float2(lx, ly);
    const float2 uf = make_float2((float)uhx, (float)uhy);
    s.t_u[k] = uf;
    s.t_q[k] = make_float2((float)qxx[i], (float)qxy[i]);
    s.t_qyy[k] = -(float)qxx[i];   // quasi-2D variant: Qzz = 0 until nem_set_qyy
    s.t_drho[k] = (float)(rho[i] - (double)R.rho0);
    s.t_acc[k] = make_float2((float)ax[i], (float)ay[i]);
    s.t_id[k] = i;
    s.t_img[k] = make_int2((int)ix, (int)iy);
    atomicAdd(&s.count[key], 1);
    atomicMax(&umax[r * UMAX_SLOTS + (i & (UMAX_SLOTS - 1))], __float_as_uint(sqrtf(uf.x * uf.x + uf.y * uf.y)));
  }
}

// Header of work item w (layout in nem_pair.h); every thread of the workgroup
// (at least 128) calls it.
__device__ void tile_header(const HdrArgs& h, int w) {
  __shared__ int cnt[128];
  const int c = threadIdx.x;
  const int rep = h.work[2 * w], tile = h.work[2 * w + 1];
  const RepDev& R = h.reps[rep];
  const int cx0 = (tile % R.tiles_x) * h.T, cy0 = (tile / R.tiles_x) * h.T;
  const int ni = min(h.T, R.nc - cx0), nj = min(h.T, R.nc - cy0);
  const int nreg = (ni + 2) * (nj + 2);
  int s0 = 0, n = 0, rx = 0, ry = 0;
  if (c < nreg) {
    // staged cell c -> region cell (rx, ry): interior row-major, then the
    // halo's bottom row, its two side columns by row, its top row
    const int k = c - ni * nj;
    if (k < 0) { rx = c % ni + 1; ry = c / ni + 1; }
    else if (k < ni + 2) { rx = k; ry = 0; }
    else if (k < ni + 2 + 2 * nj) { const int q = k - (ni + 2); ry = q / 2 + 1; rx = (q & 1) ? ni + 1 : 0; }
    else { rx = k - (ni + 2) - 2 * nj; ry = nj + 1; }
    const int gx = (cx0 + rx - 1 + R.nc) % R.nc, gy = (cy0 + ry - 1 + R.nc) % R.nc;
    const int gc = R.cell_base + gy * R.nc + gx;
    s0 = h.cell_start[gc];
    n = max(h.cell_start[gc + 1] - s0, 0);
    if (s0 < 0 || (int64_t)s0 + n > h.ntot) { atomicOr(h.flags, ERR_RANGE); s0 = 0; n = 0; }
  }
  if (c < 128) cnt[c] = n;
  __syncthreads();
  int start = 0, S = 0, nin = 0;   // cells are few: every thread sums the counts before its own
  for (int k = 0; k < nreg; ++k) {
    const int v = cnt[k];
    if (k < c) start += v;
    if (k < ni * nj) nin += v;
    S += v;
  }
  const bool over = S > h.maxp;
  int* H = h.hdr + (size_t)w * h.ints;
  const int cells = HDR_ROWS + 2 * h.T;
  if (c == 0) { H[0] = over ? 0 : nin; H[1] = over ? 0 : S; H[2] = ni | nj << 8 | (over ? 1 << 16 : 0); H[3] = rep; 
    for (int k = 0; k < MAX_PARTS; ++k) H[HDR_WORDS + k] = KMAX / 2;
  }
  if (c < ni * nj && c % ni == 0) {   // first cell of an interior row
    H[HDR_ROWS + 2 * (c / ni)] = s0 - start;
    H[HDR_ROWS + 2 * (c / ni) + 1] = start;
  }
  if (c >= nj && c < h.T) {           // rows the tile does not have
    H[HDR_ROWS + 2 * c] = 0;
    H[HDR_ROWS + 2 * c + 1] = 0x7FFFFFFF;
  }
  if (cells + 2 * c < h.ints) {
    int2 e = make_int2(0, over ? 0 : S);
    if (c < nreg && !over) e = make_int2(s0, start | rx << 16 | ry << 20);
    H[cells + 2 * c] = e.x;
    H[cells + 2 * c + 1] = e.y;
  }
  __syncthreads();
}

__global__ __launch_bounds__(128) void k_tile_headers(HdrArgs h) {
  for (int w = blockIdx.x; w < h.nwork; w += gridDim.x) tile_header(h, w);
}

// Exclusive scan of count[0 .. n) into start[0 .. n] by one workgroup of 1024
// threads, four counts a thread and pass; clears the counts.
__device__ void block_scan_counts(int* count, int* start, int n) {
  __shared__ int wave_sum[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int run = 0;
  for (int b = 0; b < n; b += 4096) {
    const int i = b + 4 * t;
    int v[4], s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = i + q < n ? count[i + q] : 0;
      s += v[q];
    }
    int inc = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(inc, d, 64);
      if (lane >= d) inc += o;
    }
    if (lane == 63) wave_sum[wv] = inc;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (k < wv) before += wave_sum[k];
      total += wave_sum[k];
    }
    int x = run + before + inc - s;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q < n) {
        start[i + q] = x;
        count[i + q] = 0;
        x += v[q];
      }
    run += total;
    __syncthreads();
  }
  if (t == 0) start[n] = run;
}

// Rebin, first kernel: re-base every particle into the cell its offset now lies
// in (cells move by at most one per direction between rebins), copy it to the
// staging arrays, count the cells and keep the old cell starts; the workgroup
// that finishes last scans the counts (nobody waits for it).
__global__ __launch_bounds__(1024) void k_rebin_key(SortArgs s) {
  if (s.req[0] == 0u) return;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i <= s.ncells; i += gridDim.x * blockDim.x)
    s.cell_old[i] = s.cell_start[i];
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < s.ntot; k += gridDim.x * blockDim.x) {
    const int r = rep_of_particle(s.reps, s.R, k);
    const RepDev R = s.reps[r];
    const int c = s.cell[k] - R.cell_base;
    if (c < 0 || c >= R.nc * R.nc) { atomicOr(s.flags, ERR_RANGE); continue; }
    int cx = c % R.nc, cy = c / R.nc;
    const float2 o = s.off[k], lo = s.offlo[k];
    int dx = (o.x < 0.0f) ? -1 : (o.x >= R.cs ? 1 : 0);
    int dy = (o.y < 0.0f) ? -1 : (o.y >= R.cs ? 1 : 0);
    if (o.x < -R.cs || o.x >= 2.0f * R.cs || o.y < -R.cs || o.y >= 2.0f * R.cs) atomicOr(s.flags, ERR_RANGE);
    float2 nh, nl;
    {
#pragma clang fp contract(off)
      // (hi, lo) - d (cs, cs_lo), renormalised
      // TwoSum of hi - d*cs keeps the rounding error of the subtraction
      const float shx = (float)(-dx) * R.cs, slx = (float)(-dx) * R.cs_lo;
      float t = o.x + shx, bp = t - o.x;
      float e = (o.x - (t - bp)) + (shx - bp);
      float l2 = (lo.x + slx) + e;
      nh.x = t + l2; nl.x = l2 - (nh.x - t);
      const float shy = (float)(-dy) * R.cs, sly = (float)(-dy) * R.cs_lo;
      t = o.y + shy; bp = t - o.y;
      e = (o.y - (t - bp)) + (shy - bp);
      l2 = (lo.y + sly) + e;
      nh.y = t + l2; nl.y = l2 - (nh.y - t);
    }
    // crossing the periodic boundary changes the particle's image
    int2 im = s.img[k];
    if (cx + dx < 0) im.x -= 1; else if (cx + dx >= R.nc) im.x += 1;
    if (cy + dy < 0) im.y -= 1; else if (cy + dy >= R.nc) im.y += 1;
    cx = (cx + dx + R.nc) % R.nc;
    cy = (cy + dy + R.nc) % R.nc;
    const int key = R.cell_base + cy * R.nc + cx;
    s.t_key[k] = key;
    s.t_off[k] = nh;
    s.t_lo[k] = nl;
    s.t_u[k] = s.u[k];
    s.t_q[k] = s.q[k];
    s.t_qyy[k] = s.qyy[k];
    s.t_drho[k] = s.drho[k];
    s.t_acc[k] = s.acc[k];
    s.t_id[k] = s.id[k];
    s.t_img[k] = im;
    atomicAdd(&s.count[key], 1);
  }
  __shared__ int last;
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(&s.flags[FLAG_TICKET], 1u) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  block_scan_counts(s.count, s.cell_start, s.ncells);
  if (threadIdx.x == 0) s.flags[FLAG_TICKET] = 0u;
}

// Rebin, second kernel: one wave per new cell collects the cell's particles
// from the old cells around it (nothing moves further), orders them by id and
// writes them to their sorted slots; then the tile headers of the new cells.
// Two launches instead of six (key, scan, scatter, per-cell sort, gather and the
// step's bookkeeping): an empty launch costs 3-5 us, and nearly every step needs
// no rebin. 137^2 box 97.6 -> 87.8 us a step, 64^2 box 77.6 -> 70.5 us.
__global__ __launch_bounds__(256) void k_rebin_place(SortArgs s, HdrArgs h) {
  if (s.req[0] == 0u) return;
  __shared__ int s_k[4][64], s_id[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int c = blockIdx.x * 4 + wv; c < s.ncells; c += gridDim.x * 4) {
    int lo = 0, hi = s.R;   // largest r with cell_base <= c
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s.reps[mid].cell_base <= c) lo = mid; else hi = mid;
    }
    const int nc = s.reps[lo].nc, base = s.reps[lo].cell_base;
    const int cx = (c - base) % nc, cy = (c - base) / nc;
    const int b = s.cell_start[c], e = s.cell_start[c + 1];
    auto old_cell = [&](int q) { return base + ((cy + q / 3 - 1 + nc) % nc) * nc + (cx + q % 3 - 1 + nc) % nc; };
    auto put = [&](int src, int rank) {
      const int k = b + rank;
      if (k < 0 || k >= e || k >= s.ntot) { atomicOr(s.flags, ERR_RANGE); return; }
      s.off[k] = s.t_off[src];
      s.offlo[k] = s.t_lo[src];
      s.u[k] = s.t_u[src];
      s.q[k] = s.t_q[src];
      s.qyy[k] = s.t_qyy[src];
      s.drho[k] = s.t_drho[src];
      s.acc[k] = s.t_acc[src];
      s.id[k] = s.t_id[src];
      s.img[k] = s.t_img[src];
      s.cell[k] = c;
    };
    int m = 0;
    for (int q = 0; q < 9; ++q) {
      const int oc = old_cell(q);
      const int k1 = min(s.cell_old[oc + 1], s.ntot);
      for (int k0 = max(s.cell_old[oc], 0); k0 < k1; k0 += 64) {
        const int k = k0 + lane;
        const bool mine = k < k1 && s.t_key[k] == c;
        const unsigned long long bal = __ballot(mine);
        const int slot = m + __popcll(bal & ((1ull << lane) - 1ull));
        if (mine && slot < 64) { s_k[wv][slot] = k; s_id[wv][slot] = s.t_id[k]; }
        m += __popcll(bal);
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (m <= 64) {
      if (lane < m) {
        const int id = s_id[wv][lane];
        int rank = 0;
        for (int j = 0; j < m; ++j) rank += s_id[wv][j] < id ? 1 : 0;
        put(s_k[wv][lane], rank);
      }
    } else {   // an overfull cell (the next Verlet build reports it): rank against every member
      for (int q = 0; q < 9; ++q) {
        const int oc = old_cell(q);
        const int k1 = min(s.cell_old[oc + 1], s.ntot);
        for (int k = max(s.cell_old[oc], 0) + lane; k < k1; k += 64) {
          if (s.t_key[k] != c) continue;
          const int id = s.t_id[k];
          int rank = 0;
          for (int p = 0; p < 9; ++p) {
            const int od = old_cell(p);
            const int j1 = min(s.cell_old[od + 1], s.ntot);
            for (int j = max(s.cell_old[od], 0); j < j1; ++j) rank += (s.t_key[j] == c && s.t_id[j] < id) ? 1 : 0;
          }
          put(k, rank);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  for (int w = blockIdx.x; w < h.nwork; w += gridDim.x) tile_header(h, w);
}

// Exclusive scan of count[c0 .. c0+nc) into cell_start[c0 ..], offset by base;
// cell_start[c0+nc] = base + total. One workgroup of 1024 threads.
__global__ __launch_bounds__(1024) void k_scan(SortArgs s, int c0, int nc, int base) {
  __shared__ int part[1024];
  const int t = threadIdx.x;
  const int chunk = (nc + 1023) / 1024;
  const int b = min(nc, t * chunk), e = min(nc, b + chunk);
  int sum = 0;
  for (int i = b; i < e; ++i) sum += s.count[c0 + i];
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {  // Hillis-Steele inclusive scan
    int v = (t >= d) ? part[t - d] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int run = base + part[t] - sum;
  for (int i = b; i < e; ++i) {
    s.cell_start[c0 + i] = run;
    run += s.count[c0 + i];
  }
  if (t == 1023) s.cell_start[c0 + nc] = base + part[1023];
}

// Place each staged particle in its cell's range (arbitrary order inside).
__global__ void k_scatter(SortArgs s, int k0, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int k = k0 + i;
    const int key = s.t_key[k];
    if (key < 0 || key >= s.ncells) { atomicOr(s.flags, ERR_RANGE); continue; }
    const int slot = s.cell_start[key] + atomicAdd(&s.cursor[key], 1);
    if (slot < 0 || slot >= s.ntot) { atomicOr(s.flags, ERR_RANGE); continue; }
    s.perm[slot] = k;
  }
}

// Canonical order inside each cell: ascending particle id (insertion sort of
// the short per-cell runs, one thread per cell).
__global__ void k_cellsort(SortArgs s, int c0, int nc) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += gridDim.x * blockDim.x) {
    const int b = s.cell_start[c0 + i], e = s.cell_start[c0 + i + 1];
    if (b < 0 || e > s.ntot || b > e) { atomicOr(s.flags, ERR_RANGE); continue; }
    bool ok = true;
    for (int a = b; a < e; ++a) {
      const int v = s.perm[a];
      if (v < 0 || v >= s.ntot) ok = false;
    }
    if (!ok) { atomicOr(s.flags, ERR_RANGE); continue; }
    for (int a = b + 1; a < e; ++a) {
      const int v = s.perm[a];
      const int kv = s.t_id[v];
      int c = a - 1;
      while (c >= b && s.t_id[s.perm[c]] > kv) { s.perm[c + 1] = s.perm[c]; --c; }
      s.perm[c + 1] = v;
    }
  }
}

// Move staged particles to their sorted slots; clear count/cursor of the cells.
__global__ void k_gather(SortArgs s, int k0, int n, int c0, int nc) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int k = k0 + i;
    const int src = s.perm[k];
    if (src < 0 || src >= s.ntot) { atomicOr(s.flags, ERR_RANGE); continue; }
    s.off[k] = s.t_off[src];
    s.offlo[k] = s.t_lo[src];
    s.u[k] = s.t_u[src];
    s.q[k] = s.t_q[src];
    s.qyy[k] = s.t_qyy[src];
    s.drho[k] = s.t_drho[src];
    s.acc[k] = s.t_acc[src];
    s.id[k] = s.t_id[src];
    s.img[k] = s.t_img[src];
    s.cell[k] = s.t_key[src];
  }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += stride) {
    s.count[c0 + i] = 0;
    s.cursor[c0 + i] = 0;
  }
}

// Requests of the next step (parity p): a Verlet rebuild when relist is set
// (new state, tile change, restore), the rebin request kept or cleared; the
// other parity's words are cleared. order: of the list just built (LIST_NONE: as it was).
__global__ void k_set_requests(unsigned* flags, int p, int keep_rebin, int relist, unsigned order) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  if (order != LIST_NONE) flags[FLAG_ORDER] = order;
  unsigned* req = flags + FLAG_REQ;
  if (!keep_rebin) req[2 * p] = 0u;
  req[2 * p + 1] = relist ? 1u : 0u;
  req[2 * (1 - p)] = 0u;
  req[2 * (1 - p) + 1] = 0u;
}

// Position of sorted particle k at the integer time level,
// r^n = r^{n+1/2} - u^{n+1/2} dt/2, relative to the box of its image (may lie
// just outside [0, L) after the half-step back).
__device__ inline void position_n(const SortArgs& s, const RepDev& R, int k, double& x, double& y) {
#pragma clang fp contract(off)
  const int c = s.cell[k] - R.cell_base;
  const int cx = c % R.nc, cy = c / R.nc;
  const float2 o = s.off[k], lo = s.offlo[k], uh = s.u[k];
  const double hdt = 0.5 * (double)R.dt;
  x = (double)cx * R.csd + ((double)o.x + (double)lo.x) - hdt * (double)uh.x;
  y = (double)cy * R.csd + ((double)o.y + (double)lo.y) - hdt * (double)uh.y;
}

// The same wrapped into [0, L).
__device__ inline void position_n_wrapped(const SortArgs& s, const RepDev& R, int k, double& x, double& y) {
#pragma clang fp contract(off)
  position_n(s, R, k, x, y);
  x = x - R.Ld * floor(x / R.Ld); if (x >= R.Ld) x -= R.Ld;
  y = y - R.Ld * floor(y / R.Ld); if (y >= R.Ld) y -= R.Ld;
}

// Sorted state of replica r -> FP64 arrays in id order at the integer time
// level: r^n = r^{n+1/2} - u^{n+1/2} dt/2, u^n = u^{n+1/2} - a dt/2.
__global__ void k_export(SortArgs s, int r, double* out, int n) {
  const RepDev R = s.reps[r];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
#pragma clang fp contract(off)
    const int k = R.part_base + i;
    const int id = s.id[k];
    if (id < 0 || id >= n) { atomicOr(s.flags, ERR_RANGE); continue; }
    const float2 uh = s.u[k], ac = s.acc[k], q = s.q[k];
    const double hdt = 0.5 * (double)R.dt;
    const double uxn = (double)uh.x - hdt * (double)ac.x;
    const double uyn = (double)uh.y - hdt * (double)ac.y;
    double x, y;
    position_n_wrapped(s, R, k, x, y);
    out[id] = x;
    out[(size_t)n + id] = y;
    out[2 * (size_t)n + id] = uxn;
    out[3 * (size_t)n + id] = uyn;
    out[4 * (size_t)n + id] = (double)q.x;
    out[5 * (size_t)n + id] = (double)q.y;
    out[6 * (size_t)n + id] = (double)R.rho0 + (double)s.drho[k];
    out[7 * (size_t)n + id] = (double)ac.x;
    out[8 * (size_t)n + id] = (double)ac.y;
  }
}

// Cell coordinates and FP32 offsets (high part) of every particle of replica r
// at r^{n+1/2}, the values the neighbour predicate of the next step reads:
// cxy[2 id + 0/1] = cell x/y, oxy[2 id + 0/1] = offset x/y from the cell corner.
__global__ void k_export_offsets(SortArgs s, int r, int n, int* cxy, float* oxy) {
  const RepDev R = s.reps[r];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int k = R.part_base + i;
    const int id = s.id[k];
    const int c = s.cell[k] - R.cell_base;
    if (id < 0 || id >= n || c < 0 || c >= R.nc * R.nc) { atomicOr(s.flags, ERR_RANGE); continue; }
    const float2 o = s.off[k];
    cxy[2 * (size_t)id] = c % R.nc;
    cxy[2 * (size_t)id + 1] = c / R.nc;
    oxy[2 * (size_t)id] = o.x;
    oxy[2 * (size_t)id + 1] = o.y;
  }
}

// Qyy of replica r (quasi-2D variant) to or from an FP64 array in id order:
// to_device != 0 copies buf[id] into the sorted array, else the reverse.
__global__ void k_qyy_io(SortArgs s, int r, int n, double* buf, int to_device) {
  const RepDev R = s.reps[r];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int k = R.part_base + i;
    const int id = s.id[k];
    if (id < 0 || id >= n) { atomicOr(s.flags, ERR_RANGE); continue; }
    if (to_device) s.qyy[k] = (float)buf[id];
    else buf[id] = (double)s.qyy[k];
  }
}

// Pathlines: inv[id] = sorted slot of every particle of replica r.
__global__ void k_track_inv(SortArgs s, int r, int n, int* inv) {
  const RepDev R = s.reps[r];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int k = R.part_base + i;
    const int id = s.id[k];
    if (id < 0 || id >= n) { atomicOr(s.flags, ERR_RANGE); continue; }
    inv[id] = k;
  }
}

// Unwrapped integer-level positions of the particles ids[0..nt):
// out[t] = x + img_x L, out[nt + t] = y + img_y L.
__global__ void k_track(SortArgs s, int r, int n, const int* inv, const int* ids, int nt, double* out) {
  const RepDev R = s.reps[r];
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += gridDim.x * blockDim.x) {
#pragma clang fp contract(off)
    const int id = ids[t];
    const int k = (id >= 0 && id < n) ? inv[id] : -1;
    if (k < R.part_base || k >= R.part_base + n) {
      atomicOr(s.flags, ERR_RANGE);
      out[t] = NAN; out[(size_t)nt + t] = NAN;
      continue;
    }
    double x, y;
    position_n(s, R, k, x, y);
    const int2 im = s.img[k];
    out[t] = x + (double)im.x * R.Ld;
    out[(size_t)nt + t] = y + (double)im.y * R.Ld;
  }
}

// Mixing: counts[(by * B + bx) * ncol + c] = particles of colour c (by id) in
// bin (bx, by) of a B x B partition of the box, from the wrapped integer-level
// positions, bx = floor(x B / L).
__global__ void k_colour_counts(SortArgs s, int r, int n, const uint8_t* colour, int ncol, int B,
                                unsigned long long* counts) {
  const RepDev R = s.reps[r];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
#pragma clang fp contract(off)
    const int k = R.part_base + i;
    const int id = s.id[k];
    if (id < 0 || id >= n) { atomicOr(s.flags, ERR_RANGE); continue; }
    const int c = colour[id];
    if (c >= ncol) { atomicOr(s.flags, ERR_RANGE); continue; }
    double x, y;
    position_n_wrapped(s, R, k, x, y);
    const int bx = min(max((int)floor(x * (double)B / R.Ld), 0), B - 1);
    const int by = min(max((int)floor(y * (double)B / R.Ld), 0), B - 1);
    atomicAdd(&counts[((size_t)by * B + bx) * ncol + c], 1ull);
  }
}

// FP64 reductions of replica r at the integer time level (fixed grid, fixed
// tree: the result does not depend on scheduling). Stage 1: one partial per
// block in red[64 + 8*b + k]; stage 2 sums them in order into red[0..6]:
// sum ux, sum uy, sum |u|^2 / 2, max |u|, max |Q|_F, sum F_i, sum F_grad_i
// (fe = per-particle free-energy terms, ntot apart; may be NULL).
constexpr int RED_BLOCKS = 256;
__global__ __launch_bounds__(256) void k_reduce1(SortArgs s, int r, int n, const double* fe, double* red) {
  const RepDev R = s.reps[r];
  __shared__ double sh[7][256];
  double a0 = 0, a1 = 0, a2 = 0, m0 = 0, m1 = 0, f0 = 0, f1 = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int k = R.part_base + i;
    const float2 uh = s.u[k], ac = s.acc[k], q = s.q[k];
    const double hdt = 0.5 * (double)R.dt;
    const double ux = (double)uh.x - hdt * (double)ac.x, uy = (double)uh.y - hdt * (double)ac.y;
    const double u2 = ux * ux + uy * uy;
    a0 += ux; a1 += uy; a2 += 0.5 * u2;
    m0 = fmax(m0, sqrt(u2));
    if (R.q3d) {  // 3x3 Frobenius norm, Qzz = -Qxx - Qyy
      const double qa = q.x, qb = q.y, qc = s.qyy[k], qz = -qa - qc;
      m1 = fmax(m1, sqrt(qa * qa + 2.0 * qb * qb + qc * qc + qz * qz));
    } else {
      m1 = fmax(m1, sqrt(2.0 * ((double)q.x * q.x + (double)q.y * q.y)));
    }
    if (fe) { f0 += fe[k]; f1 += fe[(size_t)s.ntot + k]; }
  }
  const int t = threadIdx.x;
  sh[0][t] = a0; sh[1][t] = a1; sh[2][t] = a2; sh[3][t] = m0; sh[4][t] = m1; sh[5][t] = f0; sh[6][t] = f1;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) {
    if (t < d) {
      sh[0][t] += sh[0][t + d]; sh[1][t] += sh[1][t + d]; sh[2][t] += sh[2][t + d];
      sh[3][t] = fmax(sh[3][t], sh[3][t + d]); sh[4][t] = fmax(sh[4][t], sh[4][t + d]);
      sh[5][t] += sh[5][t + d]; sh[6][t] += sh[6][t + d];
    }
    __syncthreads();
  }
  if (t < 7) red[64 + 8 * blockIdx.x + t] = sh[t][0];
}
__global__ __launch_bounds__(256) void k_reduce2(double* red) {
  // one thread a value, in block order, on partials loaded all at once (35 us with a load before each addition)
  __shared__ double sh[RED_BLOCKS][8];
  for (int i = threadIdx.x; i < RED_BLOCKS * 8; i += 256) sh[i / 8][i % 8] = red[64 + i];
  __syncthreads();
  const int k = threadIdx.x;
  if (k >= 7) return;
  const bool most = k == 3 || k == 4;
  double v = 0.0;
#pragma unroll 8
  for (int b = 0; b < RED_BLOCKS; ++b) v = most ? fmax(v, sh[b][k]) : v + sh[b][k];
  red[k] = v;
}

// Integer-level offsets r^n = r^{n+1/2} - u^{n+1/2} dt/2 relative to the binned
// cells (FP32), for diagnostics that need the pair geometry at r^n.
__global__ void k_int_offsets(SortArgs s, float2* out) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < s.ntot; k += gridDim.x * blockDim.x) {
    const int r = rep_of_particle(s.reps, s.R, k);
    const float hdt = 0.5f * s.reps[r].dt;
    const float2 o = s.off[k], lo = s.offlo[k], u = s.u[k];
    out[k] = make_float2(o.x + (lo.x - hdt * u.x), o.y + (lo.y - hdt * u.y));
  }
}

// -------------------------------------------------------------- launchers
static int grid_for(int n) { return max(1, min((n + 255) / 256, 2048)); }

void launch_ingest(const SortArgs& s, int r, const double* in, int n, unsigned* umax, hipStream_t st) {
  hipLaunchKernelGGL(k_ingest, dim3(grid_for(n)), dim3(256), 0, st, s, r, in, n, umax);
}
void launch_rebin(const SortArgs& s, const HdrArgs& h, hipStream_t st) {
  // few workgroups: both return at once on nearly every step
  hipLaunchKernelGGL(k_rebin_key, dim3(max(1, min((s.ntot + 1023) / 1024, 256))), dim3(1024), 0, st, s);
  hipLaunchKernelGGL(k_rebin_place, dim3(max(1, min((s.ncells + 3) / 4, 1024))), dim3(256), 0, st, s, h);
}
void launch_tile_headers(const HdrArgs& h, hipStream_t st) {
  hipLaunchKernelGGL(k_tile_headers, dim3(max(1, min(h.nwork, 2048))), dim3(128), 0, st, h);
}
void launch_sort_tail(const SortArgs& s, int k0, int n, int c0, int nc, int base, hipStream_t st) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, st, s, c0, nc, base);
  hipLaunchKernelGGL(k_scatter, dim3(grid_for(n)), dim3(256), 0, st, s, k0, n);
  hipLaunchKernelGGL(k_cellsort, dim3(grid_for(nc)), dim3(256), 0, st, s, c0, nc);
  hipLaunchKernelGGL(k_gather, dim3(grid_for(max(n, nc))), dim3(256), 0, st, s, k0, n, c0, nc);
}
void launch_set_requests(unsigned* flags, int parity, int keep_rebin, int relist, unsigned order, hipStream_t st) {
  hipLaunchKernelGGL(k_set_requests, dim3(1), dim3(64), 0, st, flags, parity, keep_rebin, relist, order);
}
void launch_int_offsets(const SortArgs& s, float2* out, hipStream_t st) {
  hipLaunchKernelGGL(k_int_offsets, dim3(grid_for(s.ntot)), dim3(256), 0, st, s, out);
}
void launch_reduce(const SortArgs& s, int r, int n, const double* fe, double* red, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce1, dim3(RED_BLOCKS), dim3(256), 0, st, s, r, n, fe, red);
  hipLaunchKernelGGL(k_reduce2, dim3(1), dim3(256), 0, st, red);
}
void launch_export(const SortArgs& s, int r, double* out, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_export, dim3(grid_for(n)), dim3(256), 0, st, s, r, out, n);
}

void launch_export_offsets(const SortArgs& s, int r, int n, int* cxy, float* oxy, hipStream_t st) {
  hipLaunchKernelGGL(k_export_offsets, dim3(grid_for(n)), dim3(256), 0, st, s, r, n, cxy, oxy);
}

void launch_qyy_io(const SortArgs& s, int r, int n, double* buf, int to_device, hipStream_t st) {
  hipLaunchKernelGGL(k_qyy_io, dim3(grid_for(n)), dim3(256), 0, st, s, r, n, buf, to_device);
}

void launch_track(const SortArgs& s, int r, int n, int* inv, const int* ids, int nt, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_track_inv, dim3(grid_for(n)), dim3(256), 0, st, s, r, n, inv);
  hipLaunchKernelGGL(k_track, dim3(grid_for(nt)), dim3(256), 0, st, s, r, n, (const int*)inv, ids, nt, out);
}

void launch_colour_counts(const SortArgs& s, int r, int n, const uint8_t* colour, int ncol, int B,
                          unsigned long long* counts, hipStream_t st) {
  hipLaunchKernelGGL(k_colour_counts, dim3(grid_for(n)), dim3(256), 0, st, s, r, n, colour, ncol, B, counts);
}

}  // namespace nem

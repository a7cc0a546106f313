// nem_pair.h -- tile staging, neighbour predicate, smoothing kernels and
// compensated sums used by every pair pass (gfx950, wave64).
#pragma once
#include "nem_dev.h"

namespace nem {

// Tile geometry for a tile side of T cells. A workgroup stages the T x T
// interior cells of its tile plus a one-cell periodic halo into LDS; interior
// cells come first so that interior particles occupy LDS slots [0, nin).
// LDS particle capacity per staged cell: 24 for the quintic spline's cells
// (side >= 3h + skin = 4 dx, 16 particles on the lattice), 10 for Wendland C2's
// (side >= 2h + skin = 2.7 dx, 7.3 on the lattice), small enough that five
// workgroups of the 8 x 8 tile fit in one CU's LDS. A tile holding more sets
// ERR_OVERFLOW.
template <int T, int KERN = 0>
struct TileCfg {
  static constexpr int NSC = (T + 2) * (T + 2);
  static constexpr int MAXP = NSC * (KERN == 1 ? 10 : 24);
};

template <int T>
struct TileLDS {
  int cstart[TileCfg<T>::NSC + 1];  // prefix of staged counts (staged-cell order)
  int gstart[TileCfg<T>::NSC];      // first global particle of each staged cell
  int slot[TileCfg<T>::NSC];        // region index (lj+1)*(ni+2)+(li+1) -> staged cell
  int hdr[8];                       // ni, nj, nint, nreg
  float2 shift[16];                 // image shift of stencil direction (dx+1) | (dy+1) << 2
};

// Tile header, built by k_tile_headers whenever the cells or the tiles change
// (new state, rebin, tile option, restored state) and read by every pair pass:
//   {interior particles nin, staged particles S, ni | nj << 8 | over
//   << 16, replica, most list words of a particle of each part of the tile
//   (HDR_WORDS, set by the Verlet build; MAX_PARTS)};
//   per interior row {global index - LDS slot, first LDS slot} (the cells of an
//   interior row are contiguous in the sorted arrays);
//   per staged cell {first global particle, first LDS slot | region x << 16 |
//   region y << 20} (interior cells first, region coordinates counted from the
//   halo corner), and closing entries whose slot is S.
// A pass therefore starts loading fields one load after its launch; deriving the
// same from the work list, the replica and cell_start in every pass was a chain
// of three loads, a scan and a search per staged particle (2048^2 box 61 us a
// step more, 64^2 box 7.5 us a step more). The uniform part is read through the
// constant address space, in one scalar load: as vector loads, each row's test
// waited for a load of its own.
// A tile over the LDS capacity has nin = S = 0 (pass A raises ERR_OVERFLOW).
constexpr int HDR_ROWS = 8, HDR_WORDS = 4;
static_assert(MAX_PARTS <= HDR_ROWS - HDR_WORDS, "a word per part");
template <int T>
struct HdrCfg {
  static constexpr int NSC = (T + 2) * (T + 2);
  static constexpr int CELLS = HDR_ROWS + 2 * T;
  static constexpr int INTS = CELLS + 2 * (NSC + 2);
};
typedef const int __attribute__((address_space(4))) ConstInt;
typedef const RepDev __attribute__((address_space(4))) ConstRep;

// Staged-cell index of region cell (li, lj), li in [-1, ni], lj in [-1, nj].
__device__ inline int staged_index(int li, int lj, int ni, int nj) {
  if (li >= 0 && li < ni && lj >= 0 && lj < nj) return lj * ni + li;
  int nint = ni * nj, rank;
  if (lj == -1) rank = li + 1;
  else if (lj < nj) rank = (ni + 2) + 2 * lj + (li == -1 ? 0 : 1);
  else rank = (ni + 2) + 2 * nj + (li + 1);
  return nint + rank;
}

// Fill the tile header and cell tables; returns the replica index. Every
// thread of the workgroup must call it.
template <int T>
__device__ int tile_setup(const StepArgs& a, int w, TileLDS<T>& L, RepDev& R) {
  const int rep = a.work[2 * w];
  const int tile = a.work[2 * w + 1];
  R = a.reps[rep];
  const int tx = tile % R.tiles_x, ty = tile / R.tiles_x;
  const int cx0 = tx * T, cy0 = ty * T;
  const int ni = min(T, R.nc - cx0), nj = min(T, R.nc - cy0);
  const int nreg = (ni + 2) * (nj + 2);
  const int t = threadIdx.x;
  __shared__ int cnt[TileCfg<T>::NSC];
  if (t < nreg) {
    const int li = t % (ni + 2) - 1, lj = t / (ni + 2) - 1;
    const int st = staged_index(li, lj, ni, nj);
    const int gx = (cx0 + li + R.nc) % R.nc, gy = (cy0 + lj + R.nc) % R.nc;
    const int gc = R.cell_base + gy * R.nc + gx;
    int s0 = 0, s1 = 0;
    if (gc >= 0 && gc < a.ncells) { s0 = a.cell_start[gc]; s1 = a.cell_start[gc + 1]; }
    else atomicOr(a.flags, ERR_RANGE);
    L.slot[t] = st;
    L.gstart[st] = s0;
    cnt[st] = max(s1 - s0, 0);
  }
  if (t == 0) { L.hdr[0] = ni; L.hdr[1] = nj; L.hdr[2] = ni * nj; L.hdr[3] = nreg; }
  if (t < 16) L.shift[t] = make_float2((float)(1 - (t & 3)) * R.cs, (float)(1 - (t >> 2)) * R.cs);
  __syncthreads();
  if (t < 64) {  // wave 0: exclusive scan of up to 128 counts, two per lane
    const int i0 = 2 * t, i1 = 2 * t + 1;
    const int v0 = i0 < nreg ? cnt[i0] : 0, v1 = i1 < nreg ? cnt[i1] : 0;
    int s = v0 + v1, inc = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      int o = __shfl_up(inc, d, 64);
      if (t >= d) inc += o;
    }
    const int ex = inc - s;
    if (t == 0) L.cstart[0] = 0;
    if (i0 < nreg) L.cstart[i0 + 1] = ex + v0;
    if (i1 < nreg) L.cstart[i1 + 1] = ex + v0 + v1;
  }
  __syncthreads();
  return rep;
}

// Staged cell containing LDS slot p, searching cstart[lo..hi).
__device__ inline int find_cell(const int* cstart, int hi, int p) {
  int lo = 0;  // invariant: cstart[lo] <= p < cstart[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (cstart[mid] <= p) lo = mid; else hi = mid;
  }
  return lo;
}

// Neighbour predicate on FP32 cell-relative offsets. For j in the stencil cell
// displaced by (dx, dy) from i's cell, sx = -dx*cs, sy = -dy*cs and
//   rx = fl(fl(oix - ojx) + sx), r2 = fl(fl(rx*rx) + fl(ry*ry)),
// accepted when 0 < r2 < R2 = fl32((3h)^2). No contraction, so the decision is
// reproducible bit for bit from the documented rule.
__device__ __forceinline__ bool pair_accept(float oix, float oiy, float ojx, float ojy, float sx,
                                            float sy, float R2, float& rx, float& ry, float& r2) {
#pragma clang fp contract(off)
  const float tx = oix - ojx;
  const float ty = oiy - ojy;
  rx = tx + sx;
  ry = ty + sy;
  const float xx = rx * rx;
  const float yy = ry * ry;
  r2 = xx + yy;
  return (r2 > 0.0f) & (r2 < R2);
}

// Smoothing kernels of support kappa h (2D), selected at compile time:
//   KERN 0: quintic spline, kappa = 3 (Eq. quintic; the paper's kernel),
//   KERN 1: Wendland C2, kappa = 2, W = a2 (1 - q/2)^4 (1 + 2q), a2 = 7/(4 pi h^2).
// F = (dW/dr)/r, so that grad_i W_ij = F r_ij.
// kernel_raw returns W and F without the replica's constant factors,
// Wr = W / a2 and Fr = F / dWc: the pair loops apply a2 once per particle after
// the sum and fold dWc into a staged per-particle factor (the volume), which
// takes two multiplies out of every pair.
//   quintic:     Wr = t3^5 - 6 t2^5 + 15 t1^5, Fr = (t3^4 - 6 t2^4 + 15 t1^4) / r,
//                t_m = (m - q)_+, q = r/h (dW/dr = dWc (...), dWc = -5 a2 / h);
//   Wendland C2: Wr = (1 - q/2)^4 (1 + 2q), Fr = (1 - q/2)^3 (dWc = -5 a2 / h^2).
// r2 is positive and far above the FP32 denormal range for every accepted pair
// (particles never come within 1e-19 of each other), so the hardware
// reciprocal square root is used without the denormal rescaling of rsqrtf.
// Every listed pair has r < 3h up to rounding, so t3 needs no clamp.
struct KW { float rinv, r, W, F; };
template <int KERN>
__device__ __forceinline__ KW kernel_raw(const RepDev& R, float r2) {
  KW k;
  k.rinv = __builtin_amdgcn_rsqf(r2);
  k.r = r2 * k.rinv;
  const float b = k.r * R.hinv;   // q
  // (1 - q)_+ and (2 - q)_+ / 2 lie in [0, 1] (q >= 0), so each is one
  // instruction with the result clamp. t2 = 2 u exactly (scaling by 2 commutes
  // with rounding), so -6 t2^4 = -96 u^4 and -6 t2^5 = -192 u^4 u give the same
  // bits as the unscaled form.
  if constexpr (KERN == 0) {
    const float t3 = 3.0f - b;
    const float u = fminf(fmaxf(fmaf(-0.5f, b, 1.0f), 0.0f), 1.0f);   // (2 - q)_+ / 2
    const float t1 = fminf(fmaxf(1.0f - b, 0.0f), 1.0f);               // (1 - q)_+
    const float t3s = t3 * t3, us = u * u, t1s = t1 * t1;
    const float t34 = t3s * t3s, u4 = us * us, t14 = t1s * t1s;
    k.W = fmaf(15.0f * t14, t1, fmaf(-192.0f * u4, u, t34 * t3));
    k.F = fmaf(15.0f, t14, fmaf(-96.0f, u4, t34)) * k.rinv;
  } else {
    const float t = fminf(fmaxf(fmaf(-0.5f, b, 1.0f), 0.0f), 1.0f);
    const float t2 = t * t;
    k.W = (t2 * t2) * fmaf(2.0f, b, 1.0f);
    k.F = t2 * t;
  }
  return k;
}

// Distance classes of the list (decided at the Verlet build with the margin
// that particles may move before the next one): outer pairs stay at q > 2 (and
// apart), middle pairs at q > 1, inner pairs are the rest. A class only drops
// terms of the spline that are exactly zero for its pairs, so a pair may always
// be taken in a later class. On the h = 1.3 dx lattice 24 of 44 pairs are outer
// and 16 middle. Wendland C2 is one polynomial: its outer class only means
// that a pair cannot coincide. Every form is zero from the support on, so a
// listed pair beyond it adds nothing and needs no test.
enum { OUTER = 0, MIDDLE = 1, INNER = 2 };
struct Spline { float t3, t34, u, u4, t1, t14; };
template <int CL>
__device__ __forceinline__ Spline spline_terms(float r, float hinv) {
  Spline s;
  if constexpr (CL == OUTER) {
    s.t3 = fminf(fmaxf(fmaf(-hinv, r, 3.0f), 0.0f), 1.0f);   // 3 - q <= 1 for an outer pair
  } else {
    // the terms take one rounded q: its error then cancels between them as the
    // terms do (from r each, the errors add up: 14% more error in the gradients)
    const float q = r * hinv;
    s.t3 = fmaxf(3.0f - q, 0.0f);
    s.u = fminf(fmaxf(fmaf(-0.5f, q, 1.0f), 0.0f), 1.0f);    // (2 - q)_+ / 2
    const float b = s.u * s.u;
    s.u4 = b * b;
    if constexpr (CL == INNER) {
      s.t1 = fminf(fmaxf(1.0f - q, 0.0f), 1.0f);             // (1 - q)_+
      const float c = s.t1 * s.t1;
      s.t14 = c * c;
    }
  }
  const float a = s.t3 * s.t3;
  s.t34 = a * a;
  return s;
}

// W / a2 of a pair at distance r (hinv in the units of r).
template <int KERN, int CL>
__device__ __forceinline__ float class_w(float r, float hinv) {
  if constexpr (KERN == 0) {
    const Spline s = spline_terms<CL>(r, hinv);
    float w = s.t34 * s.t3;
    if constexpr (CL != OUTER) w = fmaf(-192.0f * s.u4, s.u, w);
    if constexpr (CL == INNER) w = fmaf(15.0f * s.t14, s.t1, w);
    return w;
  } else {
    const float t = fminf(fmaxf(fmaf(-0.5f * hinv, r, 1.0f), 0.0f), 1.0f);
    const float t2 = t * t;
    return (t2 * t2) * fmaf(2.0f * hinv, r, 1.0f);
  }
}

// (W'(r) / r) / dWc from r and 1/r.
template <int KERN, int CL>
__device__ __forceinline__ float class_f(float r, float rinv, float hinv) {
  if constexpr (KERN == 0) {
    const Spline s = spline_terms<CL>(r, hinv);
    float f = s.t34;
    if constexpr (CL != OUTER) f = fmaf(-96.0f, s.u4, f);
    if constexpr (CL == INNER) f = fmaf(15.0f, s.t14, f);
    return f * rinv;
  } else {
    const float t = fminf(fmaxf(fmaf(-0.5f * hinv, r, 1.0f), 0.0f), 1.0f);
    return (t * t) * t;
  }
}

// W(0) / a2: the self term of the kernel sums in units of a2.
template <int KERN>
constexpr float kernel_w0_raw() { return KERN == 0 ? 66.0f : 1.0f; }

// W and F with their constant factors (passes off the step's hot path).
template <int KERN>
__device__ __forceinline__ KW kernel_wf(const RepDev& R, float r2) {
  KW k = kernel_raw<KERN>(R, r2);
  k.W *= R.a2;
  k.F *= R.dWc;
  return k;
}

// W only.
template <int KERN>
__device__ __forceinline__ float kernel_w(const RepDev& R, float r2) {
  return R.a2 * kernel_raw<KERN>(R, r2).W;
}

// A pair-sum accumulator. COMP 0: plain FP32 sum. COMP 1: Kahan summation over
// short chunks of pairs (1 to 8 list words of 2 or 3 pairs): terms are added plainly
// into the chunk partial p, and at the end of the chunk p is added to the
// running sum s with its rounding error recovered exactly (Fast2Sum) and
// carried into the next chunk's partial. That is Kahan's update applied to the
// chunk sums with the compensation held in p, so it costs two registers and
// three operations per chunk. COMP 2: Kahan compensation on every pair term.
template <int COMP>
struct Acc {
  float s, c, p;
  __device__ __forceinline__ void init() { s = 0.0f; c = 0.0f; p = 0.0f; }
  __device__ __forceinline__ static void kahan(float& s_, float& c_, float x) {
    const float y = x - c_;
    const float t = s_ + y;
    c_ = (t - s_) - y;
    s_ = t;
  }
  __device__ __forceinline__ void add(float x) {
    if constexpr (COMP == 0) s += x;
    else if constexpr (COMP == 1) p += x;
    else kahan(s, c, x);
  }
  __device__ __forceinline__ void fma(float a, float b) {
    if constexpr (COMP == 0) s = fmaf(a, b, s);
    else if constexpr (COMP == 1) p = fmaf(a, b, p);
    else { const float x = a * b; kahan(s, c, x); }
  }
  __device__ __forceinline__ void end_cell() {
    if constexpr (COMP == 1) {
#pragma clang fp contract(off)
      const float t = s + p;
      p = (s - t) + p;
      s = t;
    }
  }
  // This lane's compensated value. For COMP 1, s + p is also what closing an
  // open chunk would give (its rounded sum), so none is closed before this.
  __device__ __forceinline__ float value() const {
    if constexpr (COMP == 0) return s;
    else if constexpr (COMP == 1) return s + p;
    else return s - c;
  }
};

__device__ __forceinline__ void flag(unsigned* flags, unsigned bit) { atomicOr(flags, bit); }

// Common prologue: set up the tile, check LDS capacity. Returns false when the
// workgroup has nothing to do (uniform across the workgroup).
template <int T, int KERN = 0>
__device__ __forceinline__ bool tile_begin(const StepArgs& a, int w, TileLDS<T>& L, RepDev& R, int& rep) {
  if (w >= a.nwork) return false;
  rep = tile_setup<T>(a, w, L, R);
  const int S = L.cstart[L.hdr[3]];
  if (S > TileCfg<T, KERN>::MAXP) {
    if (threadIdx.x == 0) flag(a.flags, ERR_OVERFLOW);
    return false;
  }
  return true;
}

// ------------------------------------------------------ Verlet list entries
// A list word holds EPW slots of SBITS bits (three of 10 where the tile's LDS
// capacity fits, else two of 12 in halves of 16), rotated left by 3: an entry
// masked out of the word is the byte offset of its 8-byte LDS record, one or two
// instructions. Three slots a word instead of two 16-bit entries with a
// direction code are 60 bytes of list per particle and pass on the h = 1.3 dx
// lattice instead of 88.
template <int T, int KERN>
struct ListFmt {
  static constexpr int EPW = TileCfg<T, KERN>::MAXP <= 1024 ? 3 : 2;
  static constexpr int SH = EPW == 3 ? 10 : 16;
  static constexpr uint32_t MASK = (EPW == 3 ? 0x3FFu : 0xFFFu) << 3;
  static constexpr int CHUNK = EPW == 3 ? 5 : 8;   // words per compensation chunk of pass B (15 or 16 pairs)
  static_assert(TileCfg<T, KERN>::MAXP <= 4096, "slot must fit its field");
  __device__ __forceinline__ static uint32_t pack(uint32_t slot, int i) { return slot << (SH * i); }
  __device__ __forceinline__ static uint32_t seal(uint32_t w) { return (w << 3) | (w >> 29); }
  // byte offset of entry i of word w in an array of 8-byte records
  __device__ __forceinline__ static uint32_t at(uint32_t w, int i) {
    return (i == 0 ? w : __builtin_amdgcn_alignbit(w, w, SH * i)) & MASK;
  }
};

// vcnt of a particle: its entries in bits 0-7, and for its group of 64
// consecutive particles of the tile (a wave of the one-lane walk): entries all
// of them can take as outer (bits 8-15), as outer or middle (16-23), and the
// largest count (24-31). The first two are multiples of EPW.
__device__ __forceinline__ int vc_total(uint32_t v) { return min((int)(v & 255u), KMAX); }
__device__ __forceinline__ int vc_outer(uint32_t v) { return min((int)(v >> 8 & 255u), KMAX); }
__device__ __forceinline__ int vc_middle(uint32_t v) { return min((int)(v >> 16 & 255u), KMAX); }
__device__ __forceinline__ int vc_most(uint32_t v) { return min((int)(v >> 24), KMAX); }

template <typename V>
__device__ __forceinline__ V lds_at(const V* base, uint32_t byte_offset) {
  static_assert(sizeof(V) == 8, "records of 8 bytes");
  return *(const V*)((const char*)base + byte_offset);
}

// ------------------------------------------------- pair passes: header staging
template <int T>
struct TileRef {
  ConstInt* H;
  int nin, S, ni, nj, rep, words;
  int lo, hi;   // interior particles of this part
  bool over;
  __device__ __forceinline__ TileRef(const StepArgs& a, int w, int part = 0, int parts = 1) {
    H = (ConstInt*)(a.hdr + (size_t)w * HdrCfg<T>::INTS);
    nin = H[0]; S = H[1]; ni = H[2] & 255; nj = (H[2] >> 8) & 255; over = H[2] >> 16; rep = H[3];
    words = H[HDR_WORDS + part];
    lo = part * WG;
    hi = part + 1 < parts ? min(lo + WG, nin) : nin;
  }
  __device__ __forceinline__ int2 cell(int c) const {
    return make_int2(H[HdrCfg<T>::CELLS + 2 * c], H[HdrCfg<T>::CELLS + 2 * c + 1]);
  }
  // Global index of interior particle p (= LDS slot p).
  __device__ __forceinline__ int global(int p) const {
    int d = H[HDR_ROWS];
#pragma unroll
    for (int r = 1; r < T; ++r) {
      const int dr = H[HDR_ROWS + 2 * r], pr = H[HDR_ROWS + 2 * r + 1];
      d = p >= pr ? dr : d;
    }
    return p + d;
  }
};
__device__ __forceinline__ ConstRep& rep_of_tile(const StepArgs& a, int rep) { return ((ConstRep*)a.reps)[rep]; }

// The cell tables of a tile from its header (for kernels that walk cells).
template <int T>
struct CellLDS {
  int start[HdrCfg<T>::NSC + 1];   // first LDS slot of each staged cell
  int slot[HdrCfg<T>::NSC];        // region cell y * (ni + 2) + x -> staged cell
};
template <int T>
__device__ __forceinline__ void tile_cells(const TileRef<T>& t, CellLDS<T>& L) {
  const int nreg = (t.ni + 2) * (t.nj + 2);
  const int c = threadIdx.x;
  if (c <= nreg) {
    const int2 e = t.cell(c);
    L.start[c] = e.y & 0xFFFF;
    if (c < nreg) L.slot[((e.y >> 20) & 15) * (t.ni + 2) + ((e.y >> 16) & 15)] = c;
  }
}

// Positions of the passes that need no exact neighbour decision (A, B, C): 32-bit
// integers in units of 1/fix relative to the tile's corner, fix a power of two
// for which the 2^32 units are at least 3.5 cell sides. Differences of
// neighbours are exact modulo 2^32, so a pair needs no image shift and is
// rounded once, in the conversion to float; a unit is 2^-28 dx for cells of
// 4 dx: 16 to 64 times finer than the FP32 offsets it is taken from where these
// are above half a dx, coarser below dx / 16. Two particles closer than a unit are
// coincident here (no pair); pass D, on the offsets, takes them as neighbours, and its
// APD sums grow as r^-2 there as they would in any case. Distances are in units; the
// powers of two come out of the sums at the end.
template <typename Rep>
__device__ __forceinline__ int2 fixed_position(Rep& R, float2 off, int entry) {
  const int rx = (entry >> 16) & 15, ry = (entry >> 20) & 15;
  return make_int2((int)((uint32_t)__float2int_rn(off.x * R.fix) + (uint32_t)rx * (uint32_t)R.cs_fix),
                   (int)((uint32_t)__float2int_rn(off.y * R.fix) + (uint32_t)ry * (uint32_t)R.cs_fix));
}
struct FixPair { float rx, ry, r2; };
__device__ __forceinline__ FixPair fixed_pair(int2 pi, int2 pj) {
  FixPair d;
  d.rx = (float)(int)((uint32_t)pi.x - (uint32_t)pj.x);
  d.ry = (float)(int)((uint32_t)pi.y - (uint32_t)pj.y);
  d.r2 = fmaf(d.rx, d.rx, d.ry * d.ry);
  return d;
}

// Stage every particle of the tile and its halo: LPC lanes take one cell each
// round (LPC = 16 for the quintic's cells of 16 particles, 8 for Wendland's of
// 7.3). load(g) returns a value, store(slot, entry, value) writes it to LDS; the
// first particles of all cells of a batch of rounds are loaded before any is
// stored, so their latencies overlap.
template <int T, int KERN, typename Load, typename Store>
__device__ __forceinline__ void stage_tile(const TileRef<T>& t, Load&& load, Store&& store) {
  constexpr int LPC = KERN == 1 ? 8 : 16, GR = WG / LPC, NSC = HdrCfg<T>::NSC;
  constexpr int ROUNDS = (NSC + GR - 1) / GR, BATCH = ROUNDS < 4 ? ROUNDS : 4;
  const int lane = threadIdx.x % LPC, grp = threadIdx.x / LPC;
#pragma unroll
  for (int r0 = 0; r0 < ROUNDS; r0 += BATCH) {
    int2 e[BATCH];
    int n[BATCH];
    decltype(load(0)) v[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int c = min(grp + (r0 + b) * GR, NSC);   // entries past the tile's cells are empty
      e[b] = t.cell(c);
      n[b] = (t.cell(c + 1).y & 0xFFFF) - (e[b].y & 0xFFFF);
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
      if (lane < n[b]) v[b] = load(e[b].x + lane);
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      if (lane < n[b]) store((e[b].y & 0xFFFF) + lane, e[b].y, v[b]);
      for (int k = lane + LPC; k < n[b]; k += LPC) store((e[b].y & 0xFFFF) + k, e[b].y, load(e[b].x + k));
    }
  }
}

// Global index of LDS slot t (staging loop).
template <int T>
__device__ __forceinline__ int staged_global(const StepArgs& a, const TileLDS<T>& L, int t) {
  const int st = find_cell(L.cstart, L.hdr[3], t);
  int g = L.gstart[st] + (t - L.cstart[st]);
  if (g < 0 || g >= a.ntot) { flag(a.flags, ERR_RANGE); g = 0; }
  return g;
}

// Lanes per particle for an iteration with `rem` particles left: the base
// value, doubled while the particles still fill the workgroup (at most 16).
__device__ __forceinline__ int lanes_for(int rem, int base_lpp) {
  int l = base_lpp;
  while (l < 16 && rem * l * 2 <= WG) l <<= 1;
  return l;
}

__device__ __forceinline__ float wave_sum(float v, int lpp) {
  for (int o = 1; o < lpp; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_sum_int(int v, int lpp) {
  for (int o = 1; o < lpp; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Pair geometry of an entry of a cell-ordered list (LDS slot | direction code <<
// 12; the direct search's, and the Verlet list of learned steps) through the
// neighbour predicate.
__device__ __forceinline__ bool verlet_pair(uint32_t e, const float2* shift, int jmax, const float2* s_off,
                                            float2 oi, float R2, int& j, float& rx, float& ry, float& r2) {
  j = min((int)(e & 0xFFFu), jmax);
  const float2 sh = shift[(e >> 12) & 15u];
  const float2 oj = s_off[j];
  return pair_accept(oi.x, oi.y, oj.x, oj.y, sh.x, sh.y, R2, rx, ry, r2);
}

constexpr int CELL_MAX = 48;   // particles of a cell that a search covers (more raise ERR_OVERFLOW)
constexpr unsigned long long MASK48 = (1ull << 48) - 1ull;

}  // namespace nem

// nem_passes.hip -- the four pair passes of one SPH time step on gfx950.
//
// Each workgroup owns a tile of T x T cells of one replica and stages the tile
// plus its one-cell periodic halo into LDS (particles are sorted by cell, so
// every cell is a contiguous run). Positions are FP32 offsets from the
// particle's cell corner; the periodic image shift of a stencil cell is a whole
// number of cell sides, so pair vectors keep the precision of the offsets
// anywhere in the box.
//
// Every pass walks the particle's Verlet list: the pairs of the 3 x 3 cell
// stencil closer than 3h + delta when the list was built, as LDS slots in the
// tile's staging order (each pass stages the same tile in the same order). Pass
// D, whose APD sums carry no kernel weight, and the list export put every entry
// through the exact FP32 predicate (0 < r^2 < (3h)^2); in passes A to C every
// term carries W or W', which are zero from the support on, so a listed pair
// beyond it adds nothing. Several lanes may share a particle (each takes every
// lpp-th list word; sums are combined with wave shuffles); a tile's short tail
// of particles is spread over more lanes.
//
// What bounds these passes is the number of vector instructions per pair (one
// per 2.5 to 3 cycles and SIMD, whatever its kind; square roots 8), then the
// list's bytes. So the list is ordered by distance class (nem_pair.h): 24 of the
// 44 pairs of the lattice need one of the spline's three terms, 16 two; the
// class bounds are the same for the 64 particles of a wave, so the loops are
// scalar; and positions are fixed-point where no predicate is decided, which
// takes the direction code, its decoding and its table read out of every pair.
// Vector instructions per particle of passes A, B, C, D on the 2048^2 box: 1748,
// 3522, 2103, 2382 -> 984, 2947, 1321, 1832; time 170, 321, 208, 237 -> 102, 247,
// 146, 183 us; on the 64^2 box, where a pass is one workgroup's latency, 17.1,
// 18.7, 16.8, 18.4 -> 8.7, 14.4, 10.8, 14.1 us.
//
//   pass A  Verlet list (rebuilt from the ~144 candidates of the stencil when
//           particles have moved too far); volume V_i = 1 / sum_j W_ij
//           (Eq. sphSum, self included)
//   pass B  correction tensor and B = alpha^{-1} (Eq. sphCorrectionMatrix),
//           velocity gradient and continuity (Eqs. sph1stDerivative,
//           sphContinuity), Q gradient and Laplacian, molecular field
//           (Eq. molecularfielddis), co-rotation (Eq. corotation), Q update
//           (Eq. mi), viscous and active accelerations (Eq. sphMomentum)
//   pass C  density filter (Eq. densityCorrection) and EoS (Eq. sphEos); APD
//           velocity variance (Eq. APD: u^{n+1/2} is the same as in pass B,
//           and this pass evaluates W anyway)
//   pass D  pressure term (Eq. sphMomentum), corrector, APD geometry sums and
//           displacement (Eq. APD) and the next step's predictor (Sec. 3.1),
//           fused
#include <algorithm>

#include "nem_dev.h"
#include "nem_pair.h"

namespace nem {

// The exact neighbour predicate on staged records {offset, region cell}: the
// cell difference times cs is the image shift of pair_accept's rule (-d cs,
// exact for d = -1, 0, 1), added in one rounding. Pass D and the list export
// decide with this one function; DUP: r2 > 0 is tested too.
template <bool DUP>
__device__ __forceinline__ bool neighbour(float2 oi, float2 ci, float2 oj, float2 cj, float cs, float R2, float& rx,
                                          float& ry, float& r2) {
#pragma clang fp contract(off)
  const float tx = oi.x - oj.x, ty = oi.y - oj.y;
  rx = fmaf(ci.x - cj.x, cs, tx);
  ry = fmaf(ci.y - cj.y, cs, ty);
  const float xx = rx * rx, yy = ry * ry;
  r2 = xx + yy;
  return (!DUP || r2 > 0.0f) && r2 < R2;
}
__device__ __forceinline__ float2 region_cell(int entry) {
  return make_float2((float)((entry >> 16) & 15), (float)((entry >> 20) & 15));
}

// Walk the direct search's list of particle g (two 16-bit entries a word);
// flush() closes a compensation chunk every 16 entries (the last, open chunk is
// summed by the accumulators' value()). One word is loaded ahead.
template <typename Body, typename Flush>
__device__ __forceinline__ void each_listed(const uint32_t* __restrict__ nl, int ntot, int g, int cnt, Body&& body,
                                            Flush&& flush) {
  const uint32_t* p = nl + g;
  uint32_t next = cnt > 0 ? p[0] : 0u;
  for (int k = 0; k < cnt; k += 2) {
    const uint32_t w = next;
    if (k + 2 < cnt) next = p[(size_t)(k / 2 + 1) * ntot];
    body(w & 0xFFFFu);
    if (k + 1 < cnt) body(w >> 16);
    if ((k & 15) == 14) flush();
  }
}

// One iteration of a pass over the tile's particles: this lane's particle, and
// its first 16 list words and counts, which are requested as soon as the tile
// header is known, together with the fields that are staged, and waited for
// once. (Three words in flight in a rotation made every iteration of three
// pairs wait for the word requested one iteration before: with one to four
// workgroups a CU that was most of a pass.)
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
template <int T>
struct Lane {
  int p, g, sub, lpp;   // particle (LDS slot) and its global index (-1: none), lane of the particle's lpp
  int nw;               // list words this lane may have
  uint32_t vc;
  u32x16 w;
  // word i of this lane: word sub + i lpp of the list (row m of it at vl + m ntot). The
  // address runs: a product for each row may be a multiply-add that reads the register
  // beside sub, and waits for the load that is in flight to it.
  __device__ __forceinline__ void load(const StepArgs& a, int i0) {
    const size_t stride = (size_t)lpp * (size_t)a.ntot;
    const uint32_t* q = a.vl + (size_t)sub * (size_t)a.ntot + (size_t)i0 * stride + (uint32_t)g;
#pragma unroll
    for (int i = 0; i < 16; ++i, q += stride)
      if (i0 + i < nw) w[i] = *q;
  }
  // list = false: the lists are not built yet (pass A of a step that renews them)
  __device__ __forceinline__ void begin(const StepArgs& a, const TileRef<T>& t, int base, int base_lpp, bool list = true) {
    lpp = lanes_for(t.hi - base, base_lpp);
    p = base + threadIdx.x / lpp;
    sub = threadIdx.x & (lpp - 1);
    g = p < t.hi ? t.global(p) : -1;
    nw = 0;
    vc = 0u;
    if (list) lists(a, t);
  }
  __device__ __forceinline__ void lists(const StepArgs& a, const TileRef<T>& t) {
    nw = (min(t.words, KMAX / 2) + lpp - 1) / lpp;
    if (g >= 0) {
      vc = a.vcnt[g];
      load(a, 0);
    }
  }
};

template <int CL> struct Class { static constexpr int value = CL; };

// Walk the lane's part of its particle's Verlet list; body(Class<CL>, byte
// offset of the neighbour's LDS record). One lane per particle: the class
// bounds are the same for the wave, so the loops are scalar. More lanes: every
// entry in the general form. flush() closes a compensation chunk every FLUSH
// words: every word in pass A, whose inner terms are the largest of a sum and
// come last (with 15 pairs to a chunk the volume, and with it the acceleration,
// was less exact than an uncompensated sum), 4 in passes C and D, 5 in pass B,
// where a chunk closes 17 sums.
template <int T, int KERN, int FLUSH, typename Body, typename Flush>
__device__ __forceinline__ void walk_list(const StepArgs& a, Lane<T>& l, Body&& body, Flush&& flush) {
  using F = ListFmt<T, KERN>;
  constexpr int EPW = F::EPW;
  const int cnt = vc_total(l.vc);
  const uint32_t vu = (uint32_t)__builtin_amdgcn_readfirstlane((int)l.vc);
  const int one = l.lpp == 1;
  const int wo = one ? vc_outer(vu) / EPW : 0, wm = one ? vc_middle(vu) / EPW : 0;
  const int wx = ((vc_most(vu) + EPW - 1) / EPW + l.lpp - 1) / l.lpp;   // <= l.nw, from the list alone
  int f = 0;
  auto chunk = [&]() {
    if (++f == FLUSH) {
      asm volatile("");   // a scalar branch around the sums, not selects on each of them
      flush();
      f = 0;
    }
  };
  for (int m0 = 0; m0 < wx; m0 += 16) {
    if (m0) l.load(a, m0);
    int m = m0;
    for (const int e = min(wo, m0 + 16); m < e; ++m) {
      const uint32_t x = l.w[m - m0];
#pragma unroll
      for (int i = 0; i < EPW; ++i) body(Class<OUTER>(), F::at(x, i));
      chunk();
    }
    for (const int e = min(wm, m0 + 16); m < e; ++m) {
      const uint32_t x = l.w[m - m0];
#pragma unroll
      for (int i = 0; i < EPW; ++i) body(Class<MIDDLE>(), F::at(x, i));
      chunk();
    }
    for (const int e = min(wx, m0 + 16); m < e; ++m) {
      const uint32_t x = l.w[m - m0];
      const int k = (l.sub + m * l.lpp) * EPW;
#pragma unroll
      for (int i = 0; i < EPW; ++i)
        if (k + i < cnt) body(Class<INNER>(), F::at(x, i));
      chunk();
    }
  }
}

// --------------------------------------------- direct search (diagnostics)
// Volumes and an explicit neighbour list (nl, ncnt) at given offsets, for the
// free-energy kernel of the diagnostics, which runs between steps on the
// integer-level positions. The step itself uses the Verlet list below.
// Phase 1 runs the predicate over the candidates of the nine stencil cells and
// records, per cell, one 64-bit word: the accepted particles as a mask in bits
// 0-47 (bit b = b-th particle of the cell; a cell holds at most 48), the
// cell's first LDS slot in bits 48-59 and the stencil direction code in bits
// 60-63. Phase 2 walks the accepted pairs in cell order, all lanes taking their
// k-th pair together: it sums the kernel terms and emits the list entries
// (coalesced stores), so the kernel is evaluated for accepted pairs only.

template <int T, int COMP, int KERN>
__device__ __forceinline__ void tile_pass_a(const StepArgs& a, int w) {
  __shared__ TileLDS<T> L;
  __shared__ float2 s_off[TileCfg<T, KERN>::MAXP];
  __shared__ unsigned long long s_mask[9 * WG];  // lane-private, cell-major
  static_assert(TileCfg<T, KERN>::MAXP <= 4096, "LDS slot must fit 12 bits");
  RepDev R;
  int rep;
  if (!tile_begin<T, KERN>(a, w, L, R, rep)) return;
  const int ni = L.hdr[0], nint = L.hdr[2], nreg = L.hdr[3];
  const int S = L.cstart[nreg];
  for (int t = threadIdx.x; t < S; t += WG) s_off[t] = a.off_cur[staged_global<T>(a, L, t)];
  __syncthreads();
  const int nin = L.cstart[nint];
  const int tid = threadIdx.x;
  for (int base = 0; base < nin; base += WG) {
    const int p = base + tid;
    if (p >= nin) break;
    const int st = find_cell(L.cstart, nint, p);
    const int li = st % ni, lj = st / ni;
    const float2 oi = s_off[p];
    int cnt = 0;
    bool big = false;
#pragma unroll 1
    for (int cidx = 0; cidx < 9; ++cidx) {
      const int dy = cidx / 3, dx = cidx % 3;  // direction + 1
      const int sc = L.slot[(lj + dy) * (ni + 2) + (li + dx)];
      const int j0 = L.cstart[sc];
      const int nj = L.cstart[sc + 1] - j0;
      if (nj > CELL_MAX) big = true;
      const uint32_t code = (uint32_t)dx | ((uint32_t)dy << 2);
      const float2 sh = L.shift[code];
      uint32_t mlo = 0u, mhi = 0u;
      const int n0 = min(nj, 32), n1 = min(nj, CELL_MAX);
      for (int b = 0; b < n0; ++b) {
        const float2 oj = s_off[j0 + b];
        float rx, ry, r2;
        if (pair_accept(oi.x, oi.y, oj.x, oj.y, sh.x, sh.y, R.R2, rx, ry, r2)) mlo |= 1u << b;
      }
      for (int b = 32; b < n1; ++b) {
        const float2 oj = s_off[j0 + b];
        float rx, ry, r2;
        if (pair_accept(oi.x, oi.y, oj.x, oj.y, sh.x, sh.y, R.R2, rx, ry, r2)) mhi |= 1u << (b - 32);
      }
      s_mask[cidx * WG + tid] = ((unsigned long long)code << 60) | ((unsigned long long)j0 << 48) |
                                ((unsigned long long)mhi << 32) | mlo;
      cnt += __popc(mlo) + __popc(mhi);
    }
    const int kept = min(cnt, KMAX);
    const int g = L.gstart[st] + (p - L.cstart[st]);
    if (g < 0 || g >= a.ntot) { flag(a.flags, ERR_RANGE); continue; }
    if (cnt > KMAX || big) flag(a.flags, ERR_OVERFLOW);
    Acc<COMP> sw;
    sw.init();
    int c = -1;
    unsigned long long m = 0ull, x = 0ull;
    uint32_t word = 0u;
    uint32_t* dst = a.nl + g;
    for (int k = 0; k < kept; ++k) {
      while (m == 0ull && c < 8) {
        ++c;
        x = s_mask[c * WG + tid];
        m = x & MASK48;
      }
      const uint32_t hi = (uint32_t)(x >> 48);  // code << 12 | first slot
      const int j = (int)(hi & 0xFFFu) + __builtin_ctzll(m);
      m &= m - 1ull;
      const float2 sh = L.shift[hi >> 12];
      const float2 oj = s_off[j];
      float rx, ry, r2;
      pair_accept(oi.x, oi.y, oj.x, oj.y, sh.x, sh.y, R.R2, rx, ry, r2);
      sw.add(kernel_raw<KERN>(R, r2).W);
      const uint32_t e = (uint32_t)j | (hi & 0xF000u);
      if (k & 1) dst[(size_t)(k >> 1) * a.ntot] = word | (e << 16);
      else word = e;
      if ((k & 15) == 15) sw.end_cell();
    }
    if (kept & 1) dst[(size_t)(kept >> 1) * a.ntot] = word;
    a.V[g] = 1.0f / (R.a2 * (kernel_w0_raw<KERN>() + sw.value()));
    a.ncnt[g] = kept;
  }
}

// ------------------------------------------------------------- pass A, Verlet
// The Verlet list holds every pair of the 3 x 3 stencil closer than 3h + delta
// (delta = 0.075 h) at the last build. It stays a superset of the neighbour
// set while no particle has moved more than 0.45 delta since the build (pass D
// checks and requests a rebuild, as does every rebin, new state, tile change
// or snapshot restore): a pair left out was at least 3h + delta apart, so it is
// still more than 3h + 0.1 delta apart; pairs outside the stencil are excluded
// by the rebin criterion. The same margin keeps outer pairs (beyond 2h + delta
// at the build) at q > 2 and middle pairs (beyond h + delta) at q > 1.

// Build: one sweep over the ~144 candidates of the stencil records, per cell and
// distance class, the listed ones as a mask; then all lanes take their k-th entry
// of a class together, in cell order, so that a list word is stored by the whole
// wave at once. The masks wait in nl, which only the diagnostics use, and come back
// nine registers for a class (in LDS they took a workgroup in five from the walk of
// the quintic's 8 x 8 tiles). A sweep per class that appended what it found, its
// lanes storing each at its own candidate, took 76 us on the 64^2 box and 1.03 ms on
// the 2048^2 one; this takes 41 us and 0.59 ms. Returns the most list words of a
// particle of the tile (kept in the header). Runs on the steps that need it only
// (every few thousand at the benchmark's speeds, and on every change between
// ordinary and learned steps).
template <int T, int KERN>
__device__ __forceinline__ int build_list(const StepArgs& a, const TileRef<T>& t, ConstRep& R, const CellLDS<T>& L,
                                       const int2* s_x, int w, int part) {
  using F = ListFmt<T, KERN>;
  constexpr int EPW = F::EPW;
  __shared__ int most;
  if (threadIdx.x == 0) most = 0;
  __syncthreads();
  const int ni = t.ni, nint = t.ni * t.nj, tid = threadIdx.x;
  const size_t ntot = (size_t)a.ntot;
  uint32_t* const nl = a.nl;
  unsigned* const flags = a.flags;
  for (int base = t.lo; base < t.hi; base += WG) {
    const int p = base + tid;
    const bool act = p < t.hi;
    int li = 0, lj = 0;
    int2 xi = make_int2(0, 0);
    if (act) {
      const int st = find_cell(L.start, nint, p);
      li = st % ni; lj = st / ni;
      xi = s_x[p];
    }
    const int g = act ? t.global(p) : 0;
    auto cell = [&](int q) { return L.slot[(lj + q / 3) * (ni + 2) + (li + q % 3)]; };
    // row r of the lane's masks in nl: 9 class + q, candidates 0-31 of cell q; for cells
    // with more, 27 + q the outer and middle ones and 36 + q the inner ones of candidates 32-47
    auto kept_mask = [&](int r) -> uint32_t& { return (nl + (size_t)r * ntot)[(uint32_t)g]; };
    int all = 0, no = 0, nm = 0;   // listed; outer; middle
    bool big = false;
    if (act) {
      // masks of the candidates j0..j0 + n of a cell, n <= 32; reads up to three records further
      auto sweep = [&](int j0, int n, uint32_t& mo, uint32_t& mm, uint32_t& mi) {
        mo = mm = mi = 0u;
#pragma unroll 1
        for (int b = 0; b < n; b += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float r2 = fixed_pair(xi, s_x[j0 + b + u]).r2;
            const uint32_t bit = 1u << (b + u);
            mi |= r2 < R.R2v_fix ? bit : 0u;
            mm |= r2 > R.R2m_fix ? bit : 0u;
            mo |= r2 > R.R2o_fix ? bit : 0u;
          }
        }
        mi &= 0xFFFFFFFFu >> (32 - n);   // n > 0
        const uint32_t self = (uint32_t)(p - j0);
        if (self < 32u) mi &= ~(1u << self);
        mo &= mi;
        mm &= mi & ~mo;
        mi &= ~(mo | mm);
        no += __popc(mo);
        nm += __popc(mm);
        all += __popc(mo) + __popc(mm) + __popc(mi);
      };
#pragma unroll 1
      for (int q = 0; q < 9; ++q) {
        const int sc = cell(q), j0 = L.start[sc], n = L.start[sc + 1] - j0;
        big |= n > CELL_MAX;
        uint32_t mo = 0u, mm = 0u, mi = 0u;
        if (n > 0) sweep(j0, min(n, 32), mo, mm, mi);
        kept_mask(q) = mo;
        kept_mask(9 + q) = mm;
        kept_mask(18 + q) = mi;
        if (n > 32) {
          sweep(j0 + 32, min(n, CELL_MAX) - 32, mo, mm, mi);
          kept_mask(27 + q) = mo | mm << 16;
          kept_mask(36 + q) = mi;
        }
      }
      if (all > KMAX || big) flag(flags, ERR_OVERFLOW);
    }
    const int kept = min(all, KMAX);
    // what every particle of the wave can take in a class, and the most entries
    int go = act ? min(no, kept) / EPW * EPW : 255, gm = act ? min(no + nm, kept) / EPW * EPW : 255, gx = kept;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      go = min(go, __shfl_xor(go, o, 64));
      gm = min(gm, __shfl_xor(gm, o, 64));
      gx = max(gx, __shfl_xor(gx, o, 64));
    }
    if ((tid & 63) == 0) atomicMax(&most, gx);
    if (!act) continue;
    uint32_t* dst = a.vl + g;
    uint32_t word = 0u;
    int k = 0, i = 0;
#pragma unroll 1
    for (int cl = OUTER; cl <= INNER; ++cl) {
      uint32_t cells[9];   // this class's masks of the cells still to come, the next one first
#pragma unroll
      for (int q = 0; q < 9; ++q) cells[q] = kept_mask(9 * cl + q);
      const int end = min(k + (cl == OUTER ? no : (cl == MIDDLE ? nm : all - no - nm)), KMAX);
      int q = -1, j0 = 0;
      bool high = false;   // the cell has candidates past the 32nd, still to come
      uint32_t m = 0u;
      while (k < end) {
        while (m == 0u) {   // ends: the masks hold the entries that were counted
          if (high) {
            const uint32_t x = kept_mask(cl == INNER ? 36 + q : 27 + q);
            m = cl == OUTER ? x & 0xFFFFu : (cl == MIDDLE ? x >> 16 : x);
            j0 += 32;
            high = false;
          } else {
            const int sc = cell(++q);
            j0 = L.start[sc];
            high = L.start[sc + 1] - j0 > 32;
            m = cells[0];
#pragma unroll
            for (int c = 0; c < 8; ++c) cells[c] = cells[c + 1];
          }
        }
        word |= F::pack((uint32_t)(j0 + __builtin_ctz(m)), i);
        m &= m - 1u;
        ++k;
        if (++i == EPW) {
          *dst = F::seal(word);
          dst += ntot;
          word = 0u;
          i = 0;
        }
      }
    }
    if (i) *dst = F::seal(word);
    a.vcnt[g] = (uint32_t)kept | (uint32_t)go << 8 | (uint32_t)gm << 16 | (uint32_t)gx << 24;
    a.off_build[g] = a.off_cur[g];
  }
  __syncthreads();
  const int words = (most + EPW - 1) / EPW;
  if (threadIdx.x == 0) ((int*)a.hdr)[(size_t)w * HdrCfg<T>::INTS + HDR_WORDS + part] = words;
  return words;
}

// The list when this step renews it, then the volume over its entries.
template <int T, int COMP, int KERN>
__device__ __forceinline__ void tile_pass_a_step(const StepArgs& a, int w, int part, int parts, bool renew) {
  __shared__ CellLDS<T> L;
  __shared__ int2 s_x[TileCfg<T, KERN>::MAXP + 3];   // the build reads four records at a time
  TileRef<T> t(a, w, part, parts);
  ConstRep& R = rep_of_tile(a, t.rep);
  Lane<T> l;
  l.begin(a, t, t.lo, 1, !renew);
  if (t.over && threadIdx.x == 0) flag(a.flags, ERR_OVERFLOW);
  if (renew) tile_cells<T>(t, L);
  stage_tile<T, KERN>(t, [&](int g) { return a.off_cur[g]; },
                      [&](int j, int e, float2 o) { s_x[j] = fixed_position(R, o, e); });
  __syncthreads();
  if (renew) {
    t.words = build_list<T, KERN>(a, t, R, L, s_x, w, part);
    Lane<T> n;   // a new one: l's words would hold their registers through the build
    n.begin(a, t, t.lo, 1);
    l = n;
  }
  const float hinv = R.hinv_fix;
  for (int base = t.lo; base < t.hi;) {
    base += WG / l.lpp;
    const int g = l.g;
    const int2 xi = s_x[g >= 0 ? l.p : 0];
    Acc<COMP> sw;
    sw.init();
    if (g >= 0)
    walk_list<T, KERN, 1>(a, l, [&](auto cl, uint32_t at) {
      constexpr int CL = decltype(cl)::value;
      const FixPair d = fixed_pair(xi, lds_at(s_x, at));
      if (CL == INNER && !(d.r2 > 0.0f)) return;   // coincident particles are no neighbours
      const float r = __builtin_amdgcn_sqrtf(d.r2);
      if constexpr (KERN == 0 && CL == OUTER) {
        const Spline k = spline_terms<CL>(r, hinv);
        sw.fma(k.t34, k.t3);
      } else {
        sw.add(class_w<KERN, CL>(r, hinv));   // the terms of W cancel: summed apart they cost V a bit
      }
    }, [&]() { sw.end_cell(); });
    const float sum = wave_sum(sw.value(), l.lpp);
    if (g >= 0 && l.sub == 0) a.V[g] = 1.0f / (R.a2 * (kernel_w0_raw<KERN>() + sum));
    if (base < t.hi) l.begin(a, t, base, 1);
  }
}

// ------------------------------------------------------------------ pass B
// Q3 = 1: quasi-2D variant, a 3x3 order tensor (Qxx, Qxy, Qyy stored,
// Qzz = -Qxx - Qyy) with the printed I/3 in the co-rotation and the molecular
// field; corrected momentum form without the lambda stress terms only.
template <int T, int COMP, int FORM, int EL, int KERN, int Q3>
__device__ __forceinline__ void tile_pass_b(const StepArgs& a, int w, int part, int parts) {
  static_assert(Q3 == 0 || (FORM == 0 && EL == 0), "quasi-2D: corrected form, no lambda terms");
  constexpr int MP = TileCfg<T, KERN>::MAXP;
  __shared__ int2 s_x[MP];
  __shared__ float2 s_u[MP];
  __shared__ float2 s_q[MP];
  __shared__ float s_V[MP];                  // V dW: V_j F = s_V[j] Fr
  __shared__ float s_rho[FORM == 1 ? MP : 1];
  __shared__ float s_qc[Q3 == 1 ? MP : 1];   // Qyy of the quasi-2D variant
  const TileRef<T> t(a, w, part, parts);
  ConstRep& R = rep_of_tile(a, t.rep);
  Lane<T> l;
  l.begin(a, t, t.lo, a.lpp);
  const float hinv = R.hinv_fix;
  // grad_i W_ij = dWc F r_ij per unit of r for Wendland C2 (F = (1 - q/2)^3); the
  // quintic's F holds 1/r, in which the unit cancels
  const float dW = KERN == 1 ? R.dWc * R.unfix : R.dWc;
  struct In { float2 off, u, q; float V, x; };
  stage_tile<T, KERN>(t, [&](int g) {
    return In{a.off_cur[g], a.u[g], a.q_cur[g], a.V[g], Q3 == 1 ? a.qyy_cur[g] : (FORM == 1 ? a.drho[g] : 0.0f)};
  }, [&](int j, int e, const In& v) {
    s_x[j] = fixed_position(R, v.off, e);
    s_u[j] = v.u;
    s_q[j] = v.q;
    if constexpr (Q3 == 1) s_qc[j] = v.x;
    s_V[j] = v.V * dW;
    if constexpr (FORM == 1) s_rho[j] = R.rho0 + v.x;
  });
  __syncthreads();
  for (int base = t.lo; base < t.hi;) {
    const int lpp = l.lpp, p = l.p, sub = l.sub, g = l.g;
    base += WG / lpp;
    const bool act = g >= 0;
    // raw pair sums (see the epilogue for their meaning)
    Acc<COMP> Sxx, Sxy, Syy, Gxx, Gxy, Gyx, Gyy, Qax, Qay, Qbx, Qby;
    Acc<COMP> Mxx_a, Mxy_a, Myy_a, Mxx_b, Mxy_b, Myy_b, Vsx, Vsy;
    Acc<COMP> Kc, V1x, V1y, A1x, A1y;
    Acc<COMP> Qcx, Qcy, Mxx_c, Mxy_c, Myy_c;   // quasi-2D: gradient and Laplacian sums of Qyy
    Sxx.init(); Sxy.init(); Syy.init(); Gxx.init(); Gxy.init(); Gyx.init(); Gyy.init();
    Qax.init(); Qay.init(); Qbx.init(); Qby.init();
    Mxx_a.init(); Mxy_a.init(); Myy_a.init(); Mxx_b.init(); Mxy_b.init(); Myy_b.init();
    Vsx.init(); Vsy.init();
    Kc.init(); V1x.init(); V1y.init(); A1x.init(); A1y.init();
    Qcx.init(); Qcy.init(); Mxx_c.init(); Mxy_c.init(); Myy_c.init();
    float2 ui = {0.f, 0.f}, qi = {0.f, 0.f};
    float qci = 0.f;
    float ri = 1.0f;
    if (act) {
      const int2 xi = s_x[p];
      ui = s_u[p];
      qi = s_q[p];
      if constexpr (Q3 == 1) qci = s_qc[p];
      if constexpr (FORM == 1) ri = s_rho[p];
      const float ri2inv = 1.0f / (ri * ri);
      walk_list<T, KERN, ListFmt<T, KERN>::CHUNK>(a, l, [&](auto cl, uint32_t at) {
        constexpr int CL = decltype(cl)::value;
        const FixPair d = fixed_pair(xi, lds_at(s_x, at));
        if (CL == INNER && !(d.r2 > 0.0f)) return;   // coincident particles are no neighbours
        const float rinv = __builtin_amdgcn_rsqf(d.r2);
        const float F = class_f<KERN, CL>(d.r2 * rinv, rinv, hinv);   // W'(r) per unit, over r and dWc
        const float2 uj = lds_at(s_u, at), qj = lds_at(s_q, at);
        const uint32_t at4 = at >> 1;
        const float c = *(const float*)((const char*)s_V + at4) * F;
        const float cx = c * d.rx, cy = c * d.ry;    // V_j grad_i W_ij
        const float e2 = rinv * rinv, ex = cx * e2, ey = cy * e2;
        const float txx = ex * d.rx, txy = ex * d.ry, tyy = ey * d.ry;   // V_j F r (x) r / r^2, per unit
        Sxx.fma(cx, d.rx); Sxy.fma(cx, d.ry); Syy.fma(cy, d.ry);
        const float dux = uj.x - ui.x, duy = uj.y - ui.y;
        const float dqa = qj.x - qi.x, dqb = qj.y - qi.y;
        Gxx.fma(dux, cx); Gxy.fma(dux, cy); Gyx.fma(duy, cx); Gyy.fma(duy, cy);
        Qax.fma(dqa, cx); Qay.fma(dqa, cy); Qbx.fma(dqb, cx); Qby.fma(dqb, cy);
        Mxx_a.fma(dqa, txx); Mxy_a.fma(dqa, txy); Myy_a.fma(dqa, tyy);
        Mxx_b.fma(dqb, txx); Mxy_b.fma(dqb, txy); Myy_b.fma(dqb, tyy);
        if constexpr (Q3 == 1) {
          const float dqc = *(const float*)((const char*)s_qc + at4) - qci;
          Qcx.fma(dqc, cx); Qcy.fma(dqc, cy);
          Mxx_c.fma(dqc, txx); Mxy_c.fma(dqc, txy); Myy_c.fma(dqc, tyy);
        }
        const float sv = (dux * d.rx + duy * d.ry) * -e2;  // (u_i - u_j).r_ij / r^2, per unit
        if constexpr (FORM == 0) {
          Vsx.fma(sv, cx); Vsy.fma(sv, cy);
        } else {
          const float rj = *(const float*)((const char*)s_rho + at4);
          const float Ft = dW * F;
          const float fx = Ft * d.rx, fy = Ft * d.ry;    // grad_i W_ij
          Kc.add(-(dux * fx + duy * fy));
          const float svr = sv / rj;
          V1x.fma(svr, fx); V1y.fma(svr, fy);
          const float rj2inv = 1.0f / (rj * rj);
          const float ca = qi.x * ri2inv + qj.x * rj2inv, cb = qi.y * ri2inv + qj.y * rj2inv;
          A1x.add(ca * fx + cb * fy); A1y.add(cb * fx - ca * fy);
        }
      }, [&]() {
        Sxx.end_cell(); Sxy.end_cell(); Syy.end_cell();
        Gxx.end_cell(); Gxy.end_cell(); Gyx.end_cell(); Gyy.end_cell();
        Qax.end_cell(); Qay.end_cell(); Qbx.end_cell(); Qby.end_cell();
        Mxx_a.end_cell(); Mxy_a.end_cell(); Myy_a.end_cell();
        Mxx_b.end_cell(); Mxy_b.end_cell(); Myy_b.end_cell();
        Vsx.end_cell(); Vsy.end_cell();
        if constexpr (FORM == 1) { Kc.end_cell(); V1x.end_cell(); V1y.end_cell(); A1x.end_cell(); A1y.end_cell(); }
        if constexpr (Q3 == 1) { Qcx.end_cell(); Qcy.end_cell(); Mxx_c.end_cell(); Mxy_c.end_cell(); Myy_c.end_cell(); }
      });
    }
    const float sxx = wave_sum(Sxx.value(), lpp), sxy = wave_sum(Sxy.value(), lpp), syy = wave_sum(Syy.value(), lpp);
    const float gxx = wave_sum(Gxx.value(), lpp), gxy = wave_sum(Gxy.value(), lpp);
    const float gyx = wave_sum(Gyx.value(), lpp), gyy = wave_sum(Gyy.value(), lpp);
    const float qax = wave_sum(Qax.value(), lpp), qay = wave_sum(Qay.value(), lpp);
    const float qbx = wave_sum(Qbx.value(), lpp), qby = wave_sum(Qby.value(), lpp);
    const float mxxa = wave_sum(Mxx_a.value(), lpp), mxya = wave_sum(Mxy_a.value(), lpp);
    const float myya = wave_sum(Myy_a.value(), lpp);
    const float mxxb = wave_sum(Mxx_b.value(), lpp), mxyb = wave_sum(Mxy_b.value(), lpp);
    const float myyb = wave_sum(Myy_b.value(), lpp);
    float vsx = 0.f, vsy = 0.f, kc = 0.f, v1x = 0.f, v1y = 0.f, a1x = 0.f, a1y = 0.f;
    float qcx = 0.f, qcy = 0.f, mxxc = 0.f, mxyc = 0.f, myyc = 0.f;
    if constexpr (Q3 == 1) {
      qcx = wave_sum(Qcx.value(), lpp); qcy = wave_sum(Qcy.value(), lpp);
      mxxc = wave_sum(Mxx_c.value(), lpp); mxyc = wave_sum(Mxy_c.value(), lpp); myyc = wave_sum(Myy_c.value(), lpp);
    }
    if constexpr (FORM == 0) { vsx = wave_sum(Vsx.value(), lpp); vsy = wave_sum(Vsy.value(), lpp); }
    else {
      kc = wave_sum(Kc.value(), lpp); v1x = wave_sum(V1x.value(), lpp); v1y = wave_sum(V1y.value(), lpp);
      a1x = wave_sum(A1x.value(), lpp); a1y = wave_sum(A1y.value(), lpp);
    }
    if (act && sub == 0) {
      // alpha = -sum_j V_j W'/r r_ij (x) r_ij, B = alpha^{-1}
      const float un = -R.unfix;
      const float axx = un * sxx, axy = un * sxy, ayy = un * syy;
      const float det = axx * ayy - axy * axy;
      const float nrm = axx * axx + 2.0f * axy * axy + ayy * ayy;
      float Bxx = 1.f, Bxy = 0.f, Byy = 1.f;
      if (det > 1e-12f * nrm && isfinite(det)) {
        const float id = 1.0f / det;
        Bxx = ayy * id; Bxy = -axy * id; Byy = axx * id;
      } else {
        flag(a.flags, ERR_SINGULAR);
      }
      // velocity gradient G_ab = du_a/dx_b = sum_l Gu[a][l] B^{lb}
      const float G11 = gxx * Bxx + gxy * Bxy, G12 = gxx * Bxy + gxy * Byy;
      const float G21 = gyx * Bxx + gyy * Bxy, G22 = gyx * Bxy + gyy * Byy;
      const float divu = G11 + G22;
      const float drho_n = a.drho[g];
      const float kk = (FORM == 0) ? -(R.rho0 + drho_n) * divu : R.mass * kc;
      a.dh[g] = drho_n + 0.5f * kk * R.dt;
      a.bk[g] = make_float4(Bxx, Bxy, Byy, kk);
      // corrected gradients of Qxx (a) and Qxy (b)
      const float dax = qax * Bxx + qay * Bxy, day = qax * Bxy + qay * Byy;
      const float dbx = qbx * Bxx + qby * Bxy, dby = qbx * Bxy + qby * Byy;
      // Laplacians: 2 sum_j V_j (Q_i - Q_j) (r_ij . g_ij) / r^2
      const float fx2 = -2.0f * R.fix;   // the sums hold Q_j - Q_i, per unit
      const float lapa = fx2 * (Bxx * mxxa + 2.0f * Bxy * mxya + Byy * myya);
      const float lapb = fx2 * (Bxx * mxxb + 2.0f * Bxy * mxyb + Byy * myyb);
      const float qa = qi.x, qb = qi.y;
      const float e12 = 0.5f * (G12 + G21), w12 = 0.5f * (G12 - G21);
      float Ha, Hb;
      float dcy = 0.f;   // d Qyy / dy (quasi-2D)
      if constexpr (Q3 == 0) {
        // molecular field (2D: the B term vanishes identically)
        const float trq2 = 2.0f * (qa * qa + qb * qb);
        const float cbulk = R.A + R.C * trq2;
        Ha = -cbulk * qa + R.K * lapa; Hb = -cbulk * qb + R.K * lapb;
        // co-rotation projected on symmetric traceless tensors (d = 2)
        const float QG = qa * (G11 - G22) + 2.0f * qb * e12;
        const float Sa = R.lam * (qa * divu + 0.5f * (G11 - G22)) + 2.0f * w12 * qb - 2.0f * R.lam * qa * QG;
        const float Sb = R.lam * (qb * divu + e12) - 2.0f * w12 * qa - 2.0f * R.lam * qb * QG;
        a.q_nxt[g] = make_float2(qa + (Sa + R.Gamma * Ha) * R.dt, qb + (Sb + R.Gamma * Hb) * R.dt);
      } else {
        // quasi-2D: Q = [[qa, qb, 0], [qb, qc, 0], [0, 0, qz]], qz = -qa - qc,
        // D = Q + I/3; E and W in-plane. The rate is projected on traceless
        // tensors (its trace is (2 lambda/3) div u from the weak compressibility).
        const float qc = qci, qz = -qa - qc;
        dcy = qcx * Bxy + qcy * Byy;
        const float lapc = fx2 * (Bxx * mxxc + 2.0f * Bxy * mxyc + Byy * myyc);
        const float lapz = -lapa - lapc;
        const float t2 = qa * qa + 2.0f * qb * qb + qc * qc + qz * qz;
        const float cb = R.A + R.C * t2, t3 = t2 * (1.0f / 3.0f);
        Ha = -cb * qa + R.B * (qa * qa + qb * qb - t3) + R.K * lapa;
        Hb = -cb * qb + R.B * qb * (qa + qc) + R.K * lapb;
        const float Hc = -cb * qc + R.B * (qb * qb + qc * qc - t3) + R.K * lapc;
        const float Hz = -cb * qz + R.B * (qz * qz - t3) + R.K * lapz;
        const float dxx = qa + (1.0f / 3.0f), dyy = qc + (1.0f / 3.0f), dzz = qz + (1.0f / 3.0f), dxy = qb;
        const float QG = qa * G11 + qb * (G12 + G21) + qc * G22;
        const float l2 = 2.0f * R.lam * QG;
        const float Sxx = 2.0f * R.lam * (G11 * dxx + e12 * dxy) + 2.0f * w12 * dxy - l2 * dxx;
        const float Sxy = R.lam * (e12 * (dxx + dyy) + dxy * divu) + w12 * (dyy - dxx) - l2 * dxy;
        const float Syy = 2.0f * R.lam * (e12 * dxy + G22 * dyy) - 2.0f * w12 * dxy - l2 * dyy;
        const float Szz = -l2 * dzz;
        const float mxx = Sxx + R.Gamma * Ha, mxy = Sxy + R.Gamma * Hb, myy = Syy + R.Gamma * Hc;
        const float mtr = (mxx + myy + Szz + R.Gamma * Hz) * (1.0f / 3.0f);
        a.q_nxt[g] = make_float2(qa + (mxx - mtr) * R.dt, qb + mxy * R.dt);
        a.qyy_nxt[g] = qc + (myy - mtr) * R.dt;
      }
      float apx, apy;
      if constexpr (FORM == 0) {
        const float vcx = vsx * Bxx + vsy * Bxy, vcy = vsx * Bxy + vsy * Byy;
        // div Q: (dQxx/dx + dQxy/dy, dQxy/dx + dQyy/dy), Qyy = -Qxx in d = 2
        const float divqx = dax + dby, divqy = (Q3 == 0) ? dbx - day : dbx + dcy;
        const float e8 = 8.0f * R.eta * R.fix;   // the sums are per unit
        apx = e8 * vcx - R.zeta * divqx;
        apy = e8 * vcy - R.zeta * divqy;
      } else {
        const float cv = R.mass * 8.0f * R.eta * R.fix / ri;
        apx = cv * v1x - R.zeta * R.mass * a1x;
        apy = cv * v1y - R.zeta * R.mass * a1y;
      }
      a.apart[g] = make_float2(apx, apy);
      if constexpr (EL == 1) {
        const float QH = 2.0f * (qa * Ha + qb * Hb);
        a.pi[g] = make_float2(R.lam * (2.0f * QH * qa - Ha), R.lam * (2.0f * QH * qb - Hb));
      }
      if (Q3 == 0 && a.feat) {  // learned-corrector inputs 0-9 (storage order): Q, grad u, H, density, activity
        float* f = a.feat + (size_t)g * 12;
        f[0] = qa; f[1] = qb;
        f[2] = G11; f[3] = G12; f[4] = G21; f[5] = G22;
        f[6] = Ha; f[7] = Hb;
        f[8] = drho_n * R.inv_rho0; f[9] = R.zeta;
      }
    }
    if (base < t.hi) l.begin(a, t, base, a.lpp);
  }
}

// ------------------------------------------------------------------ pass C
template <int T, int COMP, int KERN>
__device__ __forceinline__ void tile_pass_c(const StepArgs& a, int w, int part, int parts) {
  constexpr int MP = TileCfg<T, KERN>::MAXP;
  __shared__ int2 s_x[MP];
  __shared__ float s_dh[MP];
  __shared__ float2 s_u[MP];
  const TileRef<T> t(a, w, part, parts);
  ConstRep& R = rep_of_tile(a, t.rep);
  Lane<T> l;
  l.begin(a, t, t.lo, a.lpp);
  const float hinv = R.hinv_fix;
  struct In { float2 off, u; float dh; };
  stage_tile<T, KERN>(t, [&](int g) { return In{a.off_cur[g], a.u[g], a.dh[g]}; },
                      [&](int j, int e, const In& v) { s_x[j] = fixed_position(R, v.off, e); s_dh[j] = v.dh; s_u[j] = v.u; });
  __syncthreads();
  unsigned umb = 0;
  for (int k = 0; k < UMAX_SLOTS; ++k) umb = max(umb, a.umax_cur[t.rep * UMAX_SLOTS + k]);
  const float c0 = R.c0_factor * __uint_as_float(umb);
  const float pc = R.rho0 * c0 * c0 / R.gamma_eos;
  for (int base = t.lo; base < t.hi;) {
    const int lpp = l.lpp, p = l.p, sub = l.sub, g = l.g;
    base += WG / lpp;
    const bool act = g >= 0;
    Acc<COMP> sd, Wux, Wuy;   // in units of a2
    sd.init(); Wux.init(); Wuy.init();
    if (act) {
      const int2 xi = s_x[p];
      const float2 ui = s_u[p];
      walk_list<T, KERN, 4>(a, l, [&](auto cl, uint32_t at) {
        constexpr int CL = decltype(cl)::value;
        const FixPair d = fixed_pair(xi, lds_at(s_x, at));
        if (CL == INNER && !(d.r2 > 0.0f)) return;   // coincident particles are no neighbours
        const float W = class_w<KERN, CL>(__builtin_amdgcn_sqrtf(d.r2), hinv);
        const float2 uj = lds_at(s_u, at);
        sd.fma(*(const float*)((const char*)s_dh + (at >> 1)), W);
        Wux.fma(ui.x - uj.x, W); Wuy.fma(ui.y - uj.y, W);   // sum_j (u_i - u_j) W_ij
      }, [&]() { sd.end_cell(); Wux.end_cell(); Wuy.end_cell(); });
    }
    const float tot = wave_sum(sd.value(), lpp);
    const float wux = wave_sum(Wux.value(), lpp), wuy = wave_sum(Wuy.value(), lpp);
    if (act && sub == 0) {
      const float Vi = a.V[g];
      const float dhi = s_dh[p];
      // Shepard filter with the self term, written for rho - rho0
      const float shep = (Vi * R.a2) * fmaf(kernel_w0_raw<KERN>(), dhi, tot);
      const float drh = dhi - R.beta * (dhi - shep);
      const float x = drh * R.inv_rho0;
      float pw;  // (1 + x)^gamma - 1
      if (R.gamma_eos == 7.0f)
        pw = x * (7.0f + x * (21.0f + x * (35.0f + x * (35.0f + x * (21.0f + x * (7.0f + x))))));
      else
        pw = expm1f(R.gamma_eos * log1pf(x));
      const float rh = R.rho0 + drh;
      a.P[g] = pc * pw / (rh * rh);
      a.drhat[g] = drh;
      a.uv[g] = sqrtf(wux * wux + wuy * wuy) * (R.a2 * Vi);
    }
    if (base < t.hi) l.begin(a, t, base, a.lpp);
  }
}

// ------------------------------------------------------------------ pass D
// INTEG: corrector, 0 kick-drift-kick, 1 midpoint (the integrator parameter picks the variant at launch).
template <int T, int COMP, int FORM, int EL, int KERN, int INTEG>
__device__ __forceinline__ void tile_pass_d(const StepArgs& a, int w, int part, int parts) {
  constexpr int MP = TileCfg<T, KERN>::MAXP;
  // FORM 0 stages V dWc (V_j F = V_j dWc Fr); without the lambda stress it also
  // stages P V dWc, so that (P_i + P_j) V_j F = (P_i V_j + PV_j) Fr.
  constexpr bool PV = FORM == 0 && EL == 0;
  __shared__ float2 s_off[MP];
  __shared__ float2 s_cell[MP];   // region cell of the particle
  __shared__ float2 s_VP[MP];     // {V dWc, P V dWc or P}
  __shared__ float2 s_pi[EL == 1 ? MP : 1];
  __shared__ float s_wmax[WG / 64];
  const TileRef<T> t(a, w, part, parts);
  ConstRep& R = rep_of_tile(a, t.rep);
  Lane<T> l;
  l.begin(a, t, t.lo, a.lpp);
  const float hinv = R.hinv, cs = R.cs, R2 = R.R2;
  struct In { float2 off, pi; float V, P; };
  stage_tile<T, KERN>(t, [&](int g) {
    return In{a.off_cur[g], EL == 1 ? a.pi[g] : make_float2(0.f, 0.f), a.V[g], a.P[g]};
  }, [&](int j, int e, const In& v) {
    s_off[j] = v.off;
    s_cell[j] = region_cell(e);
    const float Vd = v.V * R.dWc;
    s_VP[j] = make_float2(Vd, PV ? v.P * Vd : v.P);
    if constexpr (EL == 1) s_pi[j] = v.pi;
  });
  __syncthreads();
  float umax_l = 0.0f;
  bool rebin = false, bad = false, relist = false;
  for (int base = t.lo; base < t.hi;) {
    const int lpp = l.lpp, p = l.p, sub = l.sub, g = l.g;
    base += WG / lpp;
    const bool act = g >= 0;
    Acc<COMP> Px, Py, Exx, Exy, Eyx, Eyy;
    Acc<COMP> Gx, Gy, Gr;   // APD geometry: sum r_ij / r^3, sum r
    Px.init(); Py.init(); Exx.init(); Exy.init(); Eyx.init(); Eyy.init();
    Gx.init(); Gy.init(); Gr.init();
    float2 oi = {0.f, 0.f};
    int nacc = 0;   // accepted neighbours taken by this lane
    if (act) {
      oi = s_off[p];
      const float2 ci = s_cell[p];
      const float Pi = PV ? a.P[g] : s_VP[p].y;
      float2 pii = {0.f, 0.f};
      if constexpr (EL == 1) pii = s_pi[p];
      walk_list<T, KERN, 4>(a, l, [&](auto cl, uint32_t at) {
        constexpr int CL = decltype(cl)::value;
        float rx, ry, r2;
        if (!neighbour<CL == INNER>(oi, ci, lds_at(s_off, at), lds_at(s_cell, at), cs, R2, rx, ry, r2)) return;
        ++nacc;
        const float rinv = __builtin_amdgcn_rsqf(r2), r = r2 * rinv;
        const float F = class_f<KERN, CL>(r, rinv, hinv);
        const float2 vp = lds_at(s_VP, at);
        const float c = (FORM == 0) ? vp.x * F : R.dWc * F;
        const float f = PV ? fmaf(Pi, vp.x, vp.y) * F : (Pi + vp.y) * c;
        Px.fma(f, rx); Py.fma(f, ry);
        const float r3 = rinv * rinv * rinv;
        Gx.fma(rx, r3); Gy.fma(ry, r3); Gr.add(r);
        if constexpr (EL == 1) {
          const float2 pj = lds_at(s_pi, at);
          const float cx = c * rx, cy = c * ry;
          const float dpa = pj.x - pii.x, dpb = pj.y - pii.y;
          Exx.fma(dpa, cx); Exy.fma(dpa, cy); Eyx.fma(dpb, cx); Eyy.fma(dpb, cy);
        }
      }, [&]() {
        Px.end_cell(); Py.end_cell(); Gx.end_cell(); Gy.end_cell(); Gr.end_cell();
        if constexpr (EL == 1) { Exx.end_cell(); Exy.end_cell(); Eyx.end_cell(); Eyy.end_cell(); }
      });
    }
    const float prx = wave_sum(Px.value(), lpp), pry = wave_sum(Py.value(), lpp);
    const float gx = wave_sum(Gx.value(), lpp), gy = wave_sum(Gy.value(), lpp), gr = wave_sum(Gr.value(), lpp);
    const int cnt = wave_sum_int(nacc, lpp);
    float exx = 0.f, exy = 0.f, eyx = 0.f, eyy = 0.f;
    if constexpr (EL == 1) {
      exx = wave_sum(Exx.value(), lpp); exy = wave_sum(Exy.value(), lpp);
      eyx = wave_sum(Eyx.value(), lpp); eyy = wave_sum(Eyy.value(), lpp);
    }
    if (act && sub == 0) {
      const float4 bk = a.bk[g];
      const float drh = a.drhat[g];
      const float rh = R.rho0 + drh;
      const float2 ap = a.apart[g];
      float ax, ay;
      if constexpr (FORM == 0) {
        ax = -rh * (prx * bk.x + pry * bk.y) + ap.x / rh;
        ay = -rh * (prx * bk.y + pry * bk.z) + ap.y / rh;
        if constexpr (EL == 1) {
          const float dPax = exx * bk.x + exy * bk.y, dPay = exx * bk.y + exy * bk.z;
          const float dPbx = eyx * bk.x + eyy * bk.y, dPby = eyx * bk.y + eyy * bk.z;
          ax += (dPax + dPby) / rh;
          ay += (dPbx - dPay) / rh;
        }
      } else {
        ax = -R.mass * prx + ap.x;
        ay = -R.mass * pry + ap.y;
      }
      const float2 uh = a.u[g];
      const float hdt = 0.5f * R.dt;
      float u1x, u1y;                                              // u^{n+1}
      if constexpr (INTEG == 0) {                                  // kick-drift-kick
        u1x = uh.x + hdt * ax; u1y = uh.y + hdt * ay;
      } else {                                                     // midpoint: u^n + a dt,
        const float2 ap = a.acc[g];                                // u^n = u^{n+1/2} - a^{n-1/2} dt/2
        u1x = (uh.x - hdt * ap.x) + R.dt * ax;
        u1y = (uh.y - hdt * ap.y) + R.dt * ay;
      }
      float drx = 0.f, dry = 0.f;
      if (R.apd && cnt > 0) {
        const float r0 = gr / (float)cnt;   // mean neighbour distance
        const float f = r0 * r0 * a.uv[g] * R.dt;
        drx = f * gx; dry = f * gy;
      }
      if (a.feat) {   // learned-corrector inputs 10-11: the step's change of acceleration a^{n+1/2} - a^{n-1/2}
        const float2 ao = a.acc[g];
        float* f = a.feat + (size_t)g * 12;
        f[10] = ax - ao.x; f[11] = ay - ao.y;
      }
      const float unx = u1x + hdt * ax, uny = u1y + hdt * ay;      // u^{n+3/2}
      // r^{n+1} - r^{n+1/2}: u^{n+1} dt/2 (kick-drift-kick) or u^{n+1/2} dt/2
      // (midpoint, r^n + u^{n+1/2} dt), then the next predictor's u^{n+3/2} dt/2
      const float vdx = INTEG == 0 ? u1x : uh.x, vdy = INTEG == 0 ? u1y : uh.y;
      const float hvx = hdt * vdx, hvy = hdt * vdy, hnx = hdt * unx, hny = hdt * uny;
      const float dispx = (hvx + hnx) + drx, dispy = (hvy + hny) + dry;
      // compensated position update: (hi, lo) += disp
      const float2 lo = a.offlo[g];
      float2 nh, nl;
      {
#pragma clang fp contract(off)
        float s = oi.x + dispx, bp = s - oi.x;
        float e = (oi.x - (s - bp)) + (dispx - bp);
        float l2 = lo.x + e;
        nh.x = s + l2; nl.x = l2 - (nh.x - s);
        s = oi.y + dispy; bp = s - oi.y;
        e = (oi.y - (s - bp)) + (dispy - bp);
        l2 = lo.y + e;
        nh.y = s + l2; nl.y = l2 - (nh.y - s);
      }
      const float dn = drh + hdt * bk.w;
      const float2 ob = a.off_build[g];
      const float bx = nh.x - ob.x, by = nh.y - ob.y;
      if (bx * bx + by * by > R.disp2) relist = true;
      a.off_nxt[g] = nh;
      a.offlo[g] = nl;
      a.u[g] = make_float2(unx, uny);
      a.acc[g] = make_float2(ax, ay);
      a.drho[g] = dn;
      umax_l = fmaxf(umax_l, sqrtf(unx * unx + uny * uny));
      if (nh.x < -R.skin_half || nh.x > R.cs + R.skin_half || nh.y < -R.skin_half || nh.y > R.cs + R.skin_half)
        rebin = true;
      if (!(isfinite(unx) && isfinite(uny) && isfinite(nh.x) && isfinite(nh.y) && isfinite(dn))) bad = true;
    }
    if (base < t.hi) l.begin(a, t, base, a.lpp);
  }
  // max speed: wave shuffles, LDS across waves, one atomic per workgroup into
  // one of UMAX_SLOTS slots of the replica (pass C takes the max of the slots)
  for (int o = 1; o < 64; o <<= 1) umax_l = fmaxf(umax_l, __shfl_xor(umax_l, o, 64));
  if ((threadIdx.x & 63) == 0) s_wmax[threadIdx.x >> 6] = umax_l;
  __syncthreads();
  if (threadIdx.x == 0) {
    float m = 0.0f;
    for (int w = 0; w < WG / 64; ++w) m = fmaxf(m, s_wmax[w]);
    if (m > 0.0f) atomicMax(&a.umax_nxt[t.rep * UMAX_SLOTS + (w & (UMAX_SLOTS - 1))], __float_as_uint(m));
  }
  if (rebin) atomicOr(&a.req_nxt[0], 1u);
  if (relist) atomicOr(&a.req_nxt[1], 1u);
  if (bad) flag(a.flags, ERR_NUMERIC);
}

// ------------------------------------------------------- free energy (FP64)
// Per-particle contributions to the free energy of Eq. freeenergy at the
// integer time level, with the elastic part written through the discrete
// Laplacian (F) and through squared corrected gradients (F_grad):
//   F_i    = V_i [A/2 trQ^2 + C/4 (trQ^2)^2 - K/2 Q:lapQ]
//   F_grad = V_i [A/2 trQ^2 + C/4 (trQ^2)^2 + K/2 sum_abc (d_c Q_ab)^2]
// (trQ^3 = 0 in 2D). Runs after the direct search on the integer-level offsets
// and walks its list (every entry passes the predicate again, as in the passes).
template <int T, int KERN>
__global__ __launch_bounds__(WG) void k_free_energy(const StepArgs a, double* fe) {
  __shared__ TileLDS<T> L;
  constexpr int MP = TileCfg<T, KERN>::MAXP;
  __shared__ float2 s_off[MP];
  __shared__ float2 s_q[MP];
  __shared__ float s_V[MP];
  __shared__ float s_qc[MP];   // Qyy (quasi-2D variant)
  RepDev R;
  int rep;
  if (!tile_begin<T, KERN>(a, blockIdx.x, L, R, rep)) return;
  const int nint = L.hdr[2], nreg = L.hdr[3];
  const int S = L.cstart[nreg];
  for (int t = threadIdx.x; t < S; t += WG) {
    const int g = staged_global<T>(a, L, t);
    s_off[t] = a.off_cur[g];
    s_q[t] = a.q_cur[g];
    s_V[t] = a.V[g];
    if (R.q3d) s_qc[t] = a.qyy_cur[g];
  }
  __syncthreads();
  const int nin = L.cstart[nint];
  for (int p = threadIdx.x; p < nin; p += WG) {
    const int st = find_cell(L.cstart, nint, p);
    const int g = L.gstart[st] + (p - L.cstart[st]);
    if (g < 0 || g >= a.ntot) { flag(a.flags, ERR_RANGE); continue; }
    const float2 oi = s_off[p], qi = s_q[p];
    Acc<1> Sxx, Sxy, Syy, Qax, Qay, Qbx, Qby, Mxxa, Mxya, Myya, Mxxb, Mxyb, Myyb;
    Acc<1> Qcx, Qcy, Mxxc, Mxyc, Myyc;
    Sxx.init(); Sxy.init(); Syy.init(); Qax.init(); Qay.init(); Qbx.init(); Qby.init();
    Mxxa.init(); Mxya.init(); Myya.init(); Mxxb.init(); Mxyb.init(); Myyb.init();
    Qcx.init(); Qcy.init(); Mxxc.init(); Mxyc.init(); Myyc.init();
    const float qci = R.q3d ? s_qc[p] : 0.0f;
    each_listed(a.nl, a.ntot, g, min(a.ncnt[g], KMAX), [&](uint32_t e) {
      int j; float rx, ry, r2;
      if (!verlet_pair(e, L.shift, S - 1, s_off, oi, R.R2, j, rx, ry, r2)) return;
      const KW k = kernel_wf<KERN>(R, r2);
      const float c = s_V[j] * k.F, cx = c * rx, cy = c * ry;
      const float txx = cx * rx, txy = cx * ry, tyy = cy * ry;
      Sxx.add(txx); Sxy.add(txy); Syy.add(tyy);
      const float2 qj = s_q[j];
      const float dqa = qj.x - qi.x, dqb = qj.y - qi.y, e2 = k.rinv * k.rinv;
      Qax.fma(dqa, cx); Qay.fma(dqa, cy); Qbx.fma(dqb, cx); Qby.fma(dqb, cy);
      const float la = -dqa * e2, lb = -dqb * e2;
      Mxxa.fma(la, txx); Mxya.fma(la, txy); Myya.fma(la, tyy);
      Mxxb.fma(lb, txx); Mxyb.fma(lb, txy); Myyb.fma(lb, tyy);
      if (R.q3d) {
        const float dqc = s_qc[j] - qci, lc = -dqc * e2;
        Qcx.fma(dqc, cx); Qcy.fma(dqc, cy);
        Mxxc.fma(lc, txx); Mxyc.fma(lc, txy); Myyc.fma(lc, tyy);
      }
    }, [&]() {
      Sxx.end_cell(); Sxy.end_cell(); Syy.end_cell(); Qax.end_cell(); Qay.end_cell(); Qbx.end_cell();
      Qby.end_cell(); Mxxa.end_cell(); Mxya.end_cell(); Myya.end_cell(); Mxxb.end_cell(); Mxyb.end_cell();
      Myyb.end_cell(); Qcx.end_cell(); Qcy.end_cell(); Mxxc.end_cell(); Mxyc.end_cell(); Myyc.end_cell();
    });
    const float axx = -Sxx.value(), axy = -Sxy.value(), ayy = -Syy.value();
    const float det = axx * ayy - axy * axy;
    float Bxx = 1.f, Bxy = 0.f, Byy = 1.f;
    if (det > 1e-12f * (axx * axx + 2.0f * axy * axy + ayy * ayy) && isfinite(det)) {
      const float id = 1.0f / det;
      Bxx = ayy * id; Bxy = -axy * id; Byy = axx * id;
    }
    const double dax = Qax.value() * Bxx + Qay.value() * Bxy, day = Qax.value() * Bxy + Qay.value() * Byy;
    const double dbx = Qbx.value() * Bxx + Qby.value() * Bxy, dby = Qbx.value() * Bxy + Qby.value() * Byy;
    const double lapa = 2.0 * (Bxx * Mxxa.value() + 2.0f * Bxy * Mxya.value() + Byy * Myya.value());
    const double lapb = 2.0 * (Bxx * Mxxb.value() + 2.0f * Bxy * Mxyb.value() + Byy * Myyb.value());
    const double qa = qi.x, qb = qi.y;
    double bulk, qlq, g2;
    if (!R.q3d) {
      const double t2 = 2.0 * (qa * qa + qb * qb);
      bulk = 0.5 * (double)R.A * t2 + 0.25 * (double)R.C * t2 * t2;
      // Q:lapQ and sum of squared gradients over the four components of Q
      qlq = 2.0 * (qa * lapa + qb * lapb);
      g2 = 2.0 * (dax * dax + day * day + dbx * dbx + dby * dby);
    } else {
      // quasi-2D: Q = diag-block [[qa, qb], [qb, qc]] + qz e_z e_z, qz = -qa - qc
      const double qc = qci, qz = -qa - qc;
      const double dcx = Qcx.value() * Bxx + Qcy.value() * Bxy, dcy = Qcx.value() * Bxy + Qcy.value() * Byy;
      const double lapc = 2.0 * (Bxx * Mxxc.value() + 2.0f * Bxy * Mxyc.value() + Byy * Myyc.value());
      const double t2 = qa * qa + 2.0 * qb * qb + qc * qc + qz * qz;
      const double t3 = qa * qa * qa + 3.0 * qb * qb * (qa + qc) + qc * qc * qc + qz * qz * qz;
      bulk = 0.5 * (double)R.A * t2 + (double)R.B / 3.0 * t3 + 0.25 * (double)R.C * t2 * t2;
      qlq = qa * lapa + 2.0 * qb * lapb + qc * lapc + qz * (-lapa - lapc);
      const double dzx = -dax - dcx, dzy = -day - dcy;
      g2 = dax * dax + day * day + 2.0 * (dbx * dbx + dby * dby) + dcx * dcx + dcy * dcy + dzx * dzx + dzy * dzy;
    }
    const double Vi = s_V[p];
    fe[g] = Vi * (bulk - 0.5 * (double)R.K * qlq);
    fe[(size_t)a.ntot + g] = Vi * (bulk + 0.5 * (double)R.K * g2);
  }
}

void launch_free_energy(int T, int kern, const StepArgs& a, double* fe, hipStream_t s) {
  const dim3 grid(a.nwork), block(WG);
  if (kern == 1) {
    if (T == 8) hipLaunchKernelGGL((k_free_energy<8, 1>), grid, block, 0, s, a, fe);
    else hipLaunchKernelGGL((k_free_energy<4, 1>), grid, block, 0, s, a, fe);
  } else {
    if (T == 8) hipLaunchKernelGGL((k_free_energy<8, 0>), grid, block, 0, s, a, fe);
    else hipLaunchKernelGGL((k_free_energy<4, 0>), grid, block, 0, s, a, fe);
  }
}

// ---------------------------------------------------------- neighbour export
// The pairs the pair passes sum over, from the Verlet list: which = 0 keeps the entries that pass the predicate
// (neighbour(), pass D's own decision), which = 1 every entry of the list.
// mode 0 counts the entries of each particle of replica rep_only into
// cnt[id]; mode 1 writes the neighbours' ids from row_ptr[id] on.
template <int T, int KERN>
__global__ __launch_bounds__(WG) void k_list_export(const StepArgs a, int rep_only, int which, int mode, int* cnt,
                                                    const int64_t* row_ptr, int32_t* col, int64_t cap) {
  constexpr int MP = TileCfg<T, KERN>::MAXP;
  __shared__ float2 s_off[MP];
  __shared__ float2 s_cell[MP];
  __shared__ int s_id[MP];
  TileRef<T> t(a, blockIdx.x);
  t.words = KMAX / 2;
  if (t.rep != rep_only) return;
  ConstRep& R = rep_of_tile(a, t.rep);
  const int nin = t.nin;
  struct In { float2 off; int id; };
  stage_tile<T, KERN>(t, [&](int g) { return In{a.off_cur[g], a.id[g]}; },
                      [&](int j, int e, const In& v) { s_off[j] = v.off; s_cell[j] = region_cell(e); s_id[j] = v.id; });
  __syncthreads();
  Lane<T> l;
  for (int p0 = 0; p0 < nin; p0 += WG) {
    const int p = p0 + threadIdx.x;
    l.p = p; l.lpp = 1; l.sub = 0; l.g = p < nin ? t.global(p) : -1;
    if (l.g < 0) continue;
    l.lists(a, t);
    l.vc = vc_total(l.vc) | (uint32_t)KMAX << 24;   // every entry in the general form: the waves here are not the passes' own
    const int idi = s_id[p];
    if (idi < 0 || idi >= R.n) { flag(a.flags, ERR_RANGE); continue; }
    const float2 oi = s_off[p], ci = s_cell[p];
    int c = 0;
    const int64_t base = (mode == 1) ? row_ptr[idi] : 0;
    walk_list<T, KERN, 1>(a, l, [&](auto, uint32_t at) {
      float rx, ry, r2;
      const bool in = neighbour<true>(oi, ci, lds_at(s_off, at), lds_at(s_cell, at), R.cs, R.R2, rx, ry, r2);
      if (which == 0 && !in) return;
      if (mode == 1) {
        if (base + c < cap) col[base + c] = s_id[at >> 3];
        else flag(a.flags, ERR_RANGE);
      }
      ++c;
    }, []() {});
    if (mode == 0) cnt[idi] = c;
  }
}

// ------------------------------------------------------- list of a checkpoint
// The passes take a distance-ordered list as the build wrote it: they test neither
// its slots nor its class bounds (a clamp is an instruction for every pair and
// pass). A list that comes from a file is tested here, once: a particle whose
// counts no build writes, or with a slot past the tile's staged particles, clears
// the list's order, and the next step renews it.
template <int T, int KERN>
__global__ __launch_bounds__(WG) void k_list_check(const StepArgs a) {
  using F = ListFmt<T, KERN>;
  const TileRef<T> t(a, blockIdx.x);
  for (int base = 0; base < t.nin; base += WG) {
    const int p = base + threadIdx.x;   // a wave is a group of 64 consecutive particles
    if (p >= t.nin) break;
    const int g = t.global(p);
    const uint32_t v = a.vcnt[g];
    const int cnt = v & 255u, no = v >> 8 & 255u, nm = v >> 16 & 255u, most = v >> 24;
    bool ok = cnt <= most && most <= KMAX && no <= nm && nm <= cnt && no % F::EPW == 0 && nm % F::EPW == 0 &&
              v >> 8 == (uint32_t)__builtin_amdgcn_readfirstlane((int)v) >> 8;
    for (int k = 0; ok && k < cnt; k += F::EPW) {
      const uint32_t x = a.vl[(size_t)(k / F::EPW) * a.ntot + g];
      for (int i = 0; i < F::EPW && k + i < cnt; ++i) ok &= (int)(F::at(x, i) >> 3) < t.S;
    }
    if (!ok) a.flags[FLAG_ORDER] = LIST_NONE;
  }
}

// ---------------------------------------------------------------- kernels
// One workgroup per tile, or fewer workgroups looping over the tiles
// (persistent launch: StepArgs::grid > 0). PARTS: blockIdx.y is the part of the tile
// (choose_parts); without, the part is a constant, which a pass of the 64^2 box is
// 0.6 us shorter for.
template <int T, int COMP, int KERN>
__global__ __launch_bounds__(WG) void k_pass_a(const StepArgs a) {
  for (int w = blockIdx.x; w < a.nwork; w += gridDim.x) { tile_pass_a<T, COMP, KERN>(a, w); __syncthreads(); }
}
// One kernel whether or not this step renews the list (the requests, where a rebin
// renews it too, or a list in the other order).
template <int T, int COMP, int KERN, bool PARTS>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(7)))
void k_pass_a_step(const StepArgs a) {
  const bool renew = (a.req_cur[0] | a.req_cur[1] | (a.flags[FLAG_ORDER] ^ LIST_BY_DISTANCE)) != 0u;   // loaded together
  for (int w = blockIdx.x; w < a.nwork; w += gridDim.x) {
    tile_pass_a_step<T, COMP, KERN>(a, w, PARTS ? blockIdx.y : 0, PARTS ? a.parts : 1, renew);
    __syncthreads();
  }
}

// Occupancy targets (waves per SIMD) of the pair passes: more resident waves
// hide the LDS and list latency in each pair's dependency chain; at its target
// no variant spills vector registers (nor does pass A at 7: most of its variants
// take 64 registers and so run 8, and a target of 8 leaves them 16 scalar registers
// fewer, which they spill).
template <int T, int COMP, int FORM, int EL, int KERN>
struct Waves {
  static constexpr int B = ((T == 4 || KERN == 1) && (COMP == 0 || (COMP == 1 && FORM == 0))) ? 5 : 1;
  static constexpr int C = 7;
  static constexpr int D = ((T == 4 || KERN == 1) && EL == 0) ? 7 : 1;
};

template <int T, int COMP, int FORM, int EL, int KERN, int Q3, bool PARTS>
__global__ __launch_bounds__(WG)
__attribute__((amdgpu_waves_per_eu(Q3 == 0 ? Waves<T, COMP, FORM, EL, KERN>::B : 1)))
void k_pass_b(const StepArgs a) {
  // the max-speed slots that this step's pass D fills (last read by the
  // previous step's pass C)
  for (int i = blockIdx.x * WG + threadIdx.x; i < a.nrep * UMAX_SLOTS; i += gridDim.x * WG) a.umax_nxt[i] = 0u;
  for (int w = blockIdx.x; w < a.nwork; w += gridDim.x) {
    tile_pass_b<T, COMP, FORM, EL, KERN, Q3>(a, w, PARTS ? blockIdx.y : 0, PARTS ? a.parts : 1);
    __syncthreads();
  }
}
template <int T, int COMP, int KERN, bool PARTS>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(Waves<T, COMP, 0, 0, KERN>::C)))
void k_pass_c(const StepArgs a) {
  if (blockIdx.x == 0 && threadIdx.x < 2) a.req_cur[threadIdx.x] = 0u;   // served
  if (blockIdx.x == 0 && threadIdx.x == 2) a.flags[FLAG_ORDER] = LIST_BY_DISTANCE;
  for (int w = blockIdx.x; w < a.nwork; w += gridDim.x) {
    tile_pass_c<T, COMP, KERN>(a, w, PARTS ? blockIdx.y : 0, PARTS ? a.parts : 1);
    __syncthreads();
  }
}
template <int T, int COMP, int FORM, int EL, int KERN, int INTEG, bool PARTS>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(Waves<T, COMP, FORM, EL, KERN>::D)))
void k_pass_d(const StepArgs a) {
  for (int w = blockIdx.x; w < a.nwork; w += gridDim.x) {
    tile_pass_d<T, COMP, FORM, EL, KERN, INTEG>(a, w, PARTS ? blockIdx.y : 0, PARTS ? a.parts : 1);
    __syncthreads();
  }
}

// ------------------------------------------------------------- dispatch
// PARTS only with the default compensation: with the others one workgroup takes a tile.
template <int T, int COMP, int FORM, int EL, int KERN, bool PARTS>
static void launch4(int pass, int q3, int integ, const StepArgs& a, hipStream_t s) {
  if constexpr (COMP == 1 && !PARTS)
    if (a.parts > 1 && pass != 1) return launch4<T, COMP, FORM, EL, KERN, true>(pass, q3, integ, a, s);
  const int full = a.grid > 0 ? std::min(a.grid, a.nwork) : a.nwork;
  const dim3 grid(full, PARTS ? a.parts : 1), block(WG);
  switch (pass) {
    case 1:
      if constexpr (!PARTS) hipLaunchKernelGGL((k_pass_a<T, COMP, KERN>), grid, block, 0, s, a);
      break;
    case 2:
      if constexpr (FORM == 0 && EL == 0) {
        if (q3) { hipLaunchKernelGGL((k_pass_b<T, COMP, 0, 0, KERN, 1, PARTS>), grid, block, 0, s, a); break; }
      }
      hipLaunchKernelGGL((k_pass_b<T, COMP, FORM, EL, KERN, 0, PARTS>), grid, block, 0, s, a);
      break;
    case 3: hipLaunchKernelGGL((k_pass_c<T, COMP, KERN, PARTS>), grid, block, 0, s, a); break;
    case 4:
      if (integ) hipLaunchKernelGGL((k_pass_d<T, COMP, FORM, EL, KERN, 1, PARTS>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_pass_d<T, COMP, FORM, EL, KERN, 0, PARTS>), grid, block, 0, s, a);
      break;
  }
}

template <int T, int COMP, int KERN>
static bool launch_phys(int pass, const PassCfg& c, const StepArgs& a, hipStream_t s) {
  if (c.Q3 && (c.FORM != 0 || c.EL != 0)) return false;
  if (c.FORM == 0 && c.EL == 0) { launch4<T, COMP, 0, 0, KERN, false>(pass, c.Q3, c.INTEG, a, s); return true; }
  if (c.FORM == 1 && c.EL == 0) { launch4<T, COMP, 1, 0, KERN, false>(pass, c.Q3, c.INTEG, a, s); return true; }
  if (c.FORM == 0 && c.EL == 1) { launch4<T, COMP, 0, 1, KERN, false>(pass, c.Q3, c.INTEG, a, s); return true; }
  return false;
}

template <int T, int KERN>
static bool launch_comp(int pass, const PassCfg& c, const StepArgs& a, hipStream_t s) {
  switch (c.COMP) {
    case 0: return launch_phys<T, 0, KERN>(pass, c, a, s);
    case 1: return launch_phys<T, 1, KERN>(pass, c, a, s);
    case 2: return launch_phys<T, 2, KERN>(pass, c, a, s);
  }
  return false;
}

template <int T, int COMP, int KERN>
static void launch_verlet(const StepArgs& a, hipStream_t s) {
  const int full = a.grid > 0 ? std::min(a.grid, a.nwork) : a.nwork;
  if constexpr (COMP == 1)
    if (a.parts > 1) {
      hipLaunchKernelGGL((k_pass_a_step<T, COMP, KERN, true>), dim3(full, a.parts), dim3(WG), 0, s, a);
      return;
    }
  hipLaunchKernelGGL((k_pass_a_step<T, COMP, KERN, false>), dim3(full), dim3(WG), 0, s, a);
}

template <int KERN>
static bool launch_verlet_k(const PassCfg& c, const StepArgs& a, hipStream_t s) {
  switch (c.COMP * 2 + (c.T == 8 ? 1 : 0)) {
    case 0: launch_verlet<4, 0, KERN>(a, s); return true;
    case 1: launch_verlet<8, 0, KERN>(a, s); return true;
    case 2: launch_verlet<4, 1, KERN>(a, s); return true;
    case 3: launch_verlet<8, 1, KERN>(a, s); return true;
    case 4: launch_verlet<4, 2, KERN>(a, s); return true;
    case 5: launch_verlet<8, 2, KERN>(a, s); return true;
  }
  return false;
}

// Pass A of a step: Verlet build (when flagged) or walk.
bool launch_pass_a_verlet(const PassCfg& c, const StepArgs& a, hipStream_t s) {
  if (c.T != 4 && c.T != 8) return false;
  if (c.KERN == 0) return launch_verlet_k<0>(c, a, s);
  if (c.KERN == 1) return launch_verlet_k<1>(c, a, s);
  return false;
}

// Tiles of 4 or 8 cells; lanes per particle (1, 2, 4) is a runtime argument.
bool launch_pass(int pass, const PassCfg& c, const StepArgs& a, hipStream_t s) {
  if (c.LPP != 1 && c.LPP != 2 && c.LPP != 4) return false;
  if (c.KERN == 0) {
    if (c.T == 4) return launch_comp<4, 0>(pass, c, a, s);
    if (c.T == 8) return launch_comp<8, 0>(pass, c, a, s);
  } else if (c.KERN == 1) {
    if (c.T == 4) return launch_comp<4, 1>(pass, c, a, s);
    if (c.T == 8) return launch_comp<8, 1>(pass, c, a, s);
  }
  return false;
}

void tile_header_shape(int T, int kern, int* maxp, int* ints) {
  *ints = T == 8 ? HdrCfg<8>::INTS : HdrCfg<4>::INTS;
  if (kern == 1) *maxp = T == 8 ? TileCfg<8, 1>::MAXP : TileCfg<4, 1>::MAXP;
  else *maxp = T == 8 ? TileCfg<8, 0>::MAXP : TileCfg<4, 0>::MAXP;
}

void launch_list_check(int T, int kern, const StepArgs& a, hipStream_t s) {
  const dim3 grid(a.nwork), block(WG);
  if (kern == 1) {
    if (T == 8) hipLaunchKernelGGL((k_list_check<8, 1>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_list_check<4, 1>), grid, block, 0, s, a);
  } else {
    if (T == 8) hipLaunchKernelGGL((k_list_check<8, 0>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_list_check<4, 0>), grid, block, 0, s, a);
  }
}

void launch_list_export(int T, int kern, const StepArgs& a, int rep, int which, int mode, int* cnt,
                        const int64_t* row_ptr, int32_t* col, int64_t cap, hipStream_t s) {
  const dim3 grid(a.nwork), block(WG);
  if (kern == 1) {
    if (T == 8) hipLaunchKernelGGL((k_list_export<8, 1>), grid, block, 0, s, a, rep, which, mode, cnt, row_ptr, col, cap);
    else hipLaunchKernelGGL((k_list_export<4, 1>), grid, block, 0, s, a, rep, which, mode, cnt, row_ptr, col, cap);
  } else {
    if (T == 8) hipLaunchKernelGGL((k_list_export<8, 0>), grid, block, 0, s, a, rep, which, mode, cnt, row_ptr, col, cap);
    else hipLaunchKernelGGL((k_list_export<4, 0>), grid, block, 0, s, a, rep, which, mode, cnt, row_ptr, col, cap);
  }
}
}  // namespace nem

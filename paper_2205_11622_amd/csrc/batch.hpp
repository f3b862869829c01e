// Device code of the batch walk of the fused SDDMM->SpMM library for gfx950:
// the kernel for any width, alignment and array size.
//
// A wave takes a merge-path slice (walker.hpp) in batches of kBatch nonzeros,
// whose columns and values it copies to LDS.  In one pass over the rows of the
// batch it forms y = b * dot(C_i, D_j) beside the columns in LDS; in a second
// pass it adds y * E_j into the rows of A.  In both passes G lanes take four
// floats each of a gathered row, so 64 / G nonzeros go side by side, and four
// such gathers are issued before the first is used: of one row, or of two or
// four short rows at once; rows of at most four nonzeros go one to a group of at
// most eight lanes.  Lane count and column tile depend on the width
// alone, at run time: every width from 1 to 256 floats takes one tile, a wider
// one equal tiles.
//
// What bounds it where columns are random is the fabric that the L2 misses go through
// (counted: 40 to 49 lines of 128 bytes a nanosecond, 120 to 160 reads outstanding in
// each channel of L2), for rows of a few nonzeros the instructions and the start of
// each wave; the 128^3 stencil reads 29 lines a nanosecond, short of both.  Measured on
// MI355X, us:
//   one nonzero at a time, one float per lane (what odd widths had) -> batch:
//     100003 power-law rows of 25, K = 100, L = 47: 604 -> 269
//     SpMM, 300007 power-law rows of 20, L = 96: 894 -> 323
//   lane groups of a wave walking rows of their own (powers of two had) -> batch:
//     150000 uniform rows of 24 at K = L = 64: 302 -> 248
//     2^17 R-MAT vertices of 20 at K = L = 16: 206 -> 93, 2^16 at 64: 126 -> 71
//     27-point stencil of 114^3 at K = L = 64: 2640 -> 1690, at 16: 1136 -> 475
//     (at 32 1075 -> 1265, 17% slower: rows of 27 fill 27 of the 32 places of a burst, and
//     the planes just outgrow L2; 100^3 967 -> 832)
//   whose groups wait for the longest row among them, and whose burst of one row
//   ends before the next begins.
// Where neighbouring rows share columns, the fabric is spared by few rows being
// walked at a time: slices of wide rows are shared by several waves (make_part).
#pragma once

#include "walker.hpp"

namespace slnr {

// Nonzeros of a batch (8 bytes of LDS each).  512 leaves occupancy to the
// registers; with 1024 (measured) widths of 64 and 100 ran 2-11% slower.
constexpr int kBatch = 512;

typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
typedef int i4_t __attribute__((ext_vector_type(4)));

// v plus the value of the 16-lane row beside it (rows 0-1, 2-3), in all lanes.
__device__ __forceinline__ float add_row16(float v) {
  const unsigned x = __builtin_bit_cast(unsigned, v);
  const u2_t r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

// v plus the value of the other half of the wave, in all lanes.
__device__ __forceinline__ float add_half(float v) {
  const unsigned x = __builtin_bit_cast(unsigned, v);
  const u2_t r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

// Sum over the G lanes of a group.
template <int G>
__device__ __forceinline__ float lanes_sum(float v) {
  if constexpr (G >= 2) v += dpp<0xB1>(v);
  if constexpr (G >= 4) v += dpp<0x4E>(v);
  if constexpr (G >= 8) v += dpp<0x141>(v);
  if constexpr (G >= 16) v += dpp<0x140>(v);
  if constexpr (G >= 32) v = add_row16(v);
  if constexpr (G >= 64) v = add_half(v);
  return v;
}

// Sum over the groups: lanes of equal (lane & (G - 1)); valid in group 0.
template <int G>
__device__ __forceinline__ float groups_sum(float v) {
  if constexpr (G <= 32) v = add_half(v);
  if constexpr (G <= 16) v = add_row16(v);
  if constexpr (G <= 4) v += dpp<0x124>(v);  // row_ror:4
  if constexpr (G <= 8) v += dpp<0x128>(v);  // row_ror:8
  return v;
}

// The two values' sums over halves: x in the lower half of the wave, y in the
// upper.
__device__ __forceinline__ float add_halves(float x, float y) {
  const u2_t r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x),
                                                  __builtin_bit_cast(unsigned, y), false, false);
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

// groups_sum of two (R = 2) or four (R = 4) values at once, each formed in the
// same order: the exchange of halves forms two of them in one instruction, that
// of 16-lane rows four, so four rows of A take 8 instructions instead of 32.
// value_of() says which value's sum a lane's part of the wave (of 64 / R lanes)
// holds, in its first G lanes.
template <int R, int G>
__device__ __forceinline__ float groups_sum_of(const float (&x)[R][4], int c) {
  static_assert(G <= 64 / R, "a group inside a part");
  float v = add_halves(x[0][c], x[1][c]);
  if constexpr (R == 4) {
    const float w = add_halves(x[2][c], x[3][c]);
    const u2_t r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v),
                                                    __builtin_bit_cast(unsigned, w), false, false);
    const unsigned lo = r[0], hi = r[1];
    v = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
  } else if constexpr (G <= 16) {
    v = add_row16(v);
  }
  if constexpr (G <= 4) v += dpp<0x124>(v);
  if constexpr (G <= 8) v += dpp<0x128>(v);
  return v;
}

template <int R>
__device__ __forceinline__ int value_of(int lane) {
  if constexpr (R == 2) return lane >> 5;
  const int k = lane >> 4;  // the 16-lane rows hold values 0, 2, 1, 3
  return ((k & 1) << 1) | (k >> 1);
}

// Floats col .. col+3 of row j; of a row too narrow for that (not `wide`) only
// the first `valid`.  `once`: with the nontemporal hint.
template <bool TAIL, bool BIG>
__device__ __forceinline__ void ld_cols(float (&r)[4], const float *base, uint32_t j, int64_t stride,
                                        int col, bool wide, int valid, bool once = false) {
  const float *p;
  if constexpr (BIG) {
    p = base + (int64_t)j * stride + col;
  } else {
    const uint32_t off = __umul24(j, (uint32_t)stride * 4u) + (uint32_t)col * 4u;
    p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + off);
  }
  if (!TAIL || wide) {  // uniform
    const f4u_t *q = reinterpret_cast<const f4u_t *>(p);
    f4u_t x;
    if (once) {            // uniform
      asm volatile("");    // two loads: merged into one, they lose the hint
      x = __builtin_nontemporal_load(q);
      asm volatile("");
    } else {
      x = *q;
    }
    r[0] = x[0]; r[1] = x[1]; r[2] = x[2]; r[3] = x[3];
  } else {
    r[0] = r[1] = r[2] = r[3] = 0.f;
    if (valid > 0) r[0] = p[0];
    if (valid > 1) r[1] = p[1];
    if (valid > 2) r[2] = p[2];
  }
}

// Parts of a slice of S items: `most` (odd), or the odd number that leaves about
// kPartItems to each.  A part costs some 4 us of its wave's time in searches and
// first loads.  us at parts of 80 / 64 items and at whole slices: 1M uniform rows of
// 16 at K = L = 128 2870 / 2915 / 2744, SpMM at 256 with 1M rows of 4 918 / 1024 / 840.
// Rounded down to an odd number the 75^3 stencil at K = 16, L = 256 takes 1130 for 810.
constexpr uint32_t kPartItems = 80;

__device__ __forceinline__ uint32_t parts_of(uint32_t S, uint32_t most) {
  if (S >= most * kPartItems) return most;
  const uint32_t fit = S / kPartItems;
  return fit > 1 ? fit | 1 : 1;
}

// One wave's share of a slice: part q of its parts.
struct Part {
  uint32_t id;              // slice, and its carry slots
  uint32_t i0, p0, i1, p1;  // start and end coordinates
  bool head;               // row i0 began in an earlier slice and ends here
  bool first, last;        // part of the slice
  int head_row;            // of the first part: the slice's head row or -1
  bool active;
};

// A slice is walked in up to a.parts parts of equal length whose inner cuts move back
// to the start of their row (of a row begun in an earlier slice: to the slice's start),
// so a part needs no carry slot.  What a slice holds of a row that goes on after it
// falls to its last part, and of a row that began before it to the part in which
// that row ends.  Part q of slice s comes right before part q + 1 on an XCD.
__device__ __forceinline__ Part make_part(const WalkArgs &a) {
  Part s;
  uint32_t S, ns, items, nnz;
  slice_count(a, &S, &ns, &items, &nnz);
  const uint32_t N = (uint32_t)a.N, xcds = (uint32_t)a.xcds;
  const uint32_t per_xcd = (ns + xcds - 1) / xcds;
  const uint32_t in_xcd = blockIdx.x / xcds;
  const uint32_t parts = parts_of(S, (uint32_t)a.parts);
  const uint32_t slice = in_xcd / parts, q = in_xcd % parts;
  s.id = blockIdx.x % xcds * per_xcd + slice;
  s.active = slice < per_xcd && s.id < ns;
  s.first = q == 0;
  s.last = q + 1 == parts;
  s.head = false;
  s.head_row = -1;
  s.i0 = s.p0 = s.i1 = s.p1 = 0;
  if (!s.active) return s;
  const uint32_t d0 = s.id * S;
  const uint32_t d1 = items - d0 > S ? d0 + S : items;
  const uint32_t each = S / parts, over = S - each * parts;
  auto cut = [&](uint32_t k) {  // the start of part k: S * k / parts items into the slice
    const uint32_t d = d0 + each * k + over * k / parts;
    return d < d1 ? d : d1;
  };
  mp_search2<64>(a.rowptr, N, nnz, cut(q), cut(q + 1), &s.i0, &s.i1);
  // Row i at the start of its nonzeros, or where the slice boundary `d` cuts it:
  // boundaries split rows of more than `snap` nonzeros only (as in make_slice).
  const uint32_t snap = snap_length(S);
  auto at = [&](uint32_t i, uint32_t d) {
    if (i >= N) return nnz;
    const uint32_t r0 = a.rowptr[i], r1 = a.rowptr[i + 1];
    return r0 + i < d && r1 - r0 > snap ? d - i : r0;
  };
  s.p0 = at(s.i0, d0);
  s.p1 = at(s.i1, s.last ? d1 : d0);
  if (s.i0 < N && s.p0 > (uint32_t)a.rowptr[s.i0]) {
    s.head = s.i0 < s.i1;
    if ((uint32_t)a.rowptr[s.i0 + 1] + s.i0 + 1 <= d1) s.head_row = (int)s.i0;
  }
  return s;
}

// What a lane wrote before, to LDS or to A, the others of the wave read after.  The memory
// operations of a wave are carried out in order, so it costs no instruction: it keeps the
// compiler from moving them past each other.
__device__ __forceinline__ void lanes_ordered() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// No row: not an index below 2^31.
constexpr uint32_t kNoRow = ~0u;

// TAIL: K or L is no multiple of 4.  BIG: 64-bit row offsets.
//
// Rows and nonzeros are counted in unsigned 32 bits: both stay below 2^31, and the
// steps past the last of them (64 rows of a window, 64 nonzeros of a burst) do not wrap.
template <int MODE, bool TAIL, bool BIG>
struct BatchWalk {
  const WalkArgs &a;
  int2 *nz;
  int lane;
  uint32_t i0, p0, i1, p1;  // the part
  bool head;
  uint32_t rlast;           // last row with a segment in the part
  float *head_slot, *tail_slot;
  uint32_t wrb;             // rowptr window: row wrb + lane covers ws .. we of the slice
  uint32_t ws, we;

  __device__ __forceinline__ BatchWalk(const WalkArgs &a_, int2 *nz_) : a(a_), nz(nz_) {}

  __device__ __forceinline__ void window(uint32_t rb) {
    if (rb == wrb) return;
    wrb = rb;
    const uint32_t r = rb + lane;
    const bool in = r <= rlast;
    const uint32_t x = in ? a.rowptr[r] : 0, y = in ? a.rowptr[r + 1] : 0;
    ws = x > p0 ? x : p0;
    we = y < p1 ? y : p1;
    if (!in) ws = we = 0;
  }

  // The rows with nonzeros s .. e-1 in the batch [pb, pe): each(row, s, n) for NPP >= 8 rows
  // at once, one a lane group, where the 64 rows of a window have at most four each
  // (groups past the last row repeat it: such rows leave a pass of the whole wave
  // mostly empty; 1M rows of 3, us: fused at 32 265 -> 219, at 16 210 -> 168, SpMM at 16
  // 145 -> 122, SDDMM at 32 139 -> 119); else several(R, rb, b, s, e)
  // for R = 4 rows rb + b[0..3] of at most NPP nonzeros or R = 2 rows of at most
  // 2 * NPP (four passes side by side either way), one(row, s, e) for the others.
  // Rows of 10 nonzeros, one after another, would leave three of the four
  // gathers of a lane unused: in sets they run 1.2-1.4x faster at K = L = 16.
  template <int NPP, typename One, typename Several, typename Each>
  __device__ __forceinline__ void for_rows(uint32_t ib, uint32_t pb, uint32_t pe, One one,
                                           Several several, Each each) {
    for (uint32_t rb = ib;; rb += 64) {
      window(rb);
      const uint32_t vs = ws > pb ? ws : pb, ve = we < pe ? we : pe;
      const int len = (int)(ve - vs);  // 0 or less: nothing of this row
      uint64_t mask = __ballot(len > 0);
      const uint64_t tall4 = __ballot(len > NPP), tall2 = __ballot(len > 2 * NPP);
      const bool more = rb + 63 < rlast && (uint32_t)__builtin_amdgcn_readlane(we, 63) < pe;
      if constexpr (NPP >= 8) {
        if (__popcll(mask) > 4 && __ballot(len > 4) == 0) {
          const int count = __popcll(mask);
          const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
          // lane k: the lane of the window's k-th row with nonzeros
          int nth = lane;
          if (mask != ~0ull) nth = __builtin_amdgcn_ds_permute((len > 0 ? rank : 63) << 2, lane);
          for (int k0 = 0; k0 < count; k0 += NPP) {
            const int k = k0 + lane / (64 / NPP);
            const int b = bperm_i(k < count ? k : count - 1, nth);
            each(rb + b, (uint32_t)bperm_i(b, (int)vs), bperm_i(b, len));
          }
          mask = 0;
        }
      }
      // the next R rows, if there are that many and none is in `tall`
      auto set = [&](auto r, uint64_t tall) {
        constexpr int R = decltype(r)::value;
        uint64_t m = mask;
#pragma unroll
        for (int u = 0; u < R - 1; ++u) m &= m - 1;
        if (m == 0) return false;
        m &= m - 1;
        if (((mask ^ m) & tall) != 0) return false;
        i4_t b, s, e;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const int i = __builtin_ctzll(mask);
          mask &= mask - 1;
          b[u] = i;
          s[u] = __builtin_amdgcn_readlane(vs, i);
          e[u] = __builtin_amdgcn_readlane(ve, i);
        }
        several(r, rb, b, s, e);
        return true;
      };
      while (mask) {
        if constexpr (NPP >= 4)
          if (set(std::integral_constant<int, 4>{}, tall4)) continue;
        if constexpr (NPP >= 2)
          if (set(std::integral_constant<int, 2>{}, tall2)) continue;
        const int b = __builtin_ctzll(mask);
        mask &= mask - 1;
        one(rb + b, __builtin_amdgcn_readlane(vs, b), __builtin_amdgcn_readlane(ve, b));
      }
      if (!more) return;
    }
  }

  // Partial dot products of the batch over floats [4 * q0, 4 * q0 + 4 * nq) of
  // the K floats: y = b * dot if `whole` (that is all of K; y holds b before),
  // else added to y.
  template <int G>
  __device__ __forceinline__ void dots(uint32_t ib, uint32_t pb, uint32_t pe, int q0, int nq, bool whole) {
    constexpr int NPP = 64 / G, U = 4;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // keeps the lane's indices out of the registers of other phases
    const int g = ln / G, q = ln & (G - 1);
    const bool lane_in = q < nq;
    const int first = 4 * (q0 + (lane_in ? q : nq - 1));  // lanes past nq repeat the last one's loads
    const int valid = a.K - first;
    // the last lane of a ragged width reads the last four floats and drops
    // those that the lane before it has: of C as of D, for an infinity in the one
    // times the other's zero would be no number
    const int col = TAIL && valid < 4 && a.K >= 4 ? a.K - 4 : first;
    const int drop = first - col;
    auto drop_front = [&](float (&x)[4]) {
      if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < 3; ++v) x[v] = v < drop ? 0.f : x[v];
      }
    };
    auto load_c = [&](float (&c)[4], uint32_t row) {
      ld_cols<TAIL, true>(c, a.C, row, a.K, col, a.K >= 4, valid, a.stream_c);
      drop_front(c);
    };
    auto load_d = [&](float (&x)[4], int j) {
      ld_cols<TAIL, BIG>(x, a.D, j, a.K, col, a.K >= 4, valid);
    };
    // all lanes of a group hold the sum and write the same word, as do the groups that
    // repeat a nonzero (all have read it by then)
    auto finish = [&](const float (&c)[4], float (&x)[4], int2 z, int2 *at) {
      drop_front(x);
      float t = 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) t = fmaf(c[v], x[v], t);
      t = lanes_sum<G>(lane_in ? t : 0.f);
      const float y = __builtin_bit_cast(float, z.y);
      at->y = __builtin_bit_cast(int, whole ? y * t : y + t);
    };
    for_rows<NPP>(
        ib, pb, pe,
        [&](uint32_t row, uint32_t s, uint32_t e) {
          float c[4];
          load_c(c, row);
          for (uint32_t k = s; k < e; k += U * NPP) {
            const int n = (int)(e - k);
            int2 *zp = nz + (k - pb);
            int2 z[U];
            float x[U][4];
            if (n >= U * NPP) {
#pragma unroll
              for (int u = 0; u < U; ++u) z[u] = zp[u * NPP + g];
#pragma unroll
              for (int u = 0; u < U; ++u) load_d(x[u], z[u].x);
              lanes_ordered();
#pragma unroll
              for (int u = 0; u < U; ++u) finish(c, x[u], z[u], zp + (u * NPP + g));
            } else {  // groups past the row's end repeat its last nonzero
              auto at = [&](int u) { return u * NPP + g < n ? u * NPP + g : n - 1; };
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (u * NPP < n) z[u] = zp[at(u)];
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (u * NPP < n) load_d(x[u], z[u].x);
              lanes_ordered();
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (u * NPP < n) finish(c, x[u], z[u], zp + at(u));
            }
          }
        },
        [&](auto r, uint32_t rb, i4_t b, i4_t s, i4_t e) {
          constexpr int R = decltype(r)::value, S = U / R;  // S passes a row
          int2 *zp[U];
          int2 z[U];
          float c[R][4], x[U][4];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int n = e[u / S] - s[u / S], k = u % S * NPP + g;
            zp[u] = nz + ((int)(s[u / S] - pb) + (k < n ? k : n - 1));
            z[u] = *zp[u];
          }
#pragma unroll
          for (int u = 0; u < R; ++u) load_c(c[u], rb + b[u]);
#pragma unroll
          for (int u = 0; u < U; ++u) load_d(x[u], z[u].x);
          lanes_ordered();
#pragma unroll
          for (int u = 0; u < U; ++u) finish(c[u / S], x[u], z[u], zp[u]);
        },
        [&](uint32_t row, uint32_t s, int n) {
          int2 *zp[U];
          int2 z[U];
          float c[4], x[U][4];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            zp[u] = nz + ((int)(s - pb) + (u < n ? u : n - 1));
            z[u] = *zp[u];
          }
          load_c(c, row);
          bool any[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            any[u] = u < 2 || __ballot(n > u) != 0;
            if (any[u]) load_d(x[u], z[u].x);
          }
          lanes_ordered();
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (any[u]) finish(c, x[u], z[u], zp[u]);
        });
  }

  __device__ __forceinline__ bool in_carry(uint32_t row) const {
    return row == i1 || (row == i0 && head);
  }

  // Where the sums of a row go (column l0 of it), also those of a first batch of it.
  __device__ __forceinline__ float *row_at(uint32_t row) const {
    return row == i1           ? tail_slot
           : row == i0 && head ? head_slot
                               : a.out + (int64_t)row * a.L + a.l0;
  }

  // Columns l0 + [4 * q0, 4 * q0 + 4 * nq) of the rows of the batch.  crow: the
  // row begun in an earlier batch of the part, or kNoRow.
  template <int G>
  __device__ __forceinline__ void rows(uint32_t ib, uint32_t pb, uint32_t pe, int q0, int nq,
                                       uint32_t crow) {
    constexpr int NPP = 64 / G, U = 4;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int g = ln / G, q = ln & (G - 1);
    const bool lane_in = q < nq;
    const int first = 4 * (q0 + (lane_in ? q : nq - 1));
    const int valid = a.Lw - first;
    // the last lane of a ragged width takes the last four columns: it forms
    // and stores the same values as its neighbour where they overlap
    const int col = TAIL && valid < 4 && a.Lw >= 4 ? a.Lw - 4 : first;
    auto load_e = [&](float (&x)[4], int j) {
      ld_cols<TAIL, BIG>(x, a.E, j, a.L, a.l0 + col, a.Lw >= 4, valid);
    };
    // A's rows carry the nontemporal hint, partial rows, which the fixup reads next, do
    // not (20000 power-law rows of 20 at 64: 50 us, 57 with it).  Rows of A, us with and
    // without: SpMM at 256 with 1M rows of 4 843 / 905, of 8 1503 / 1582.
    auto store = [&](uint32_t row, float *dst, const float (&r)[4]) {
      if (!TAIL || a.Lw >= 4) {
        f4u_t o;
        o[0] = r[0]; o[1] = r[1]; o[2] = r[2]; o[3] = r[3];
        if (in_carry(row)) {
          asm volatile("");  // two stores: merged into one, they lose the hint
          *reinterpret_cast<f4u_t *>(dst) = o;
          asm volatile("");
        } else {
          __builtin_nontemporal_store(o, reinterpret_cast<f4u_t *>(dst));
        }
      } else {
#pragma unroll
        for (int v = 0; v < 3; ++v)
          if (v < valid) dst[v] = r[v];
      }
    };
    auto add = [&](float (&acc)[4], const float (&x)[4], int2 z) {
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = fmaf(__builtin_bit_cast(float, z.y), x[v], acc[v]);
    };
    for_rows<NPP>(
        ib, pb, pe,
        [&](uint32_t row, uint32_t s, uint32_t e) {
          float acc[4] = {0.f, 0.f, 0.f, 0.f};
          // Long segments halve their rounding error by it (off the 64-bit values, without /
          // with: SpMM of power-law rows of 20 at L = 96 2.0e-7 / 1.2e-7, at 64 1.4e-7 / 1.0e-7, of 4
          // at 64 1.0e-7 / 7.8e-8, at 32 8.7e-8 / 7.5e-8) and no time: 65536 rows of 16 at K = L = 64
          // 74.2 / 74.3 us, SpMM of 1M rows of 16 at 64 612 / 612.
          const bool tall = (int)(e - s) > 2 * U * NPP;
          for (uint32_t k = s; k < e; k += U * NPP) {
            const int n = (int)(e - k);
            const int2 *zp = nz + (k - pb);
            int2 z[U];
            float x[U][4];
            if (n >= U * NPP) {
#pragma unroll
              for (int u = 0; u < U; ++u) z[u] = zp[u * NPP + g];
#pragma unroll
              for (int u = 0; u < U; ++u) load_e(x[u], z[u].x);
              if (tall) {  // uniform: the four terms first, a chain of additions a quarter as long
                float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < U; ++u) add(t, x[u], z[u]);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] += t[v];
              } else {
#pragma unroll
                for (int u = 0; u < U; ++u) add(acc, x[u], z[u]);
              }
            } else {
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (u * NPP < n) z[u] = zp[u * NPP + g < n ? u * NPP + g : n - 1];
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (u * NPP < n) load_e(x[u], z[u].x);
#pragma unroll
              for (int u = 0; u < U; ++u) {
                if ((u + 1) * NPP <= n) add(acc, x[u], z[u]);
                else if (u * NPP < n && u * NPP + g < n) add(acc, x[u], z[u]);
              }
            }
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[v] = groups_sum<G>(acc[v]);
          if (lane_in && g == 0) {
            float *dst = row_at(row) + col;
            if (row == crow) {
#pragma unroll
              for (int v = 0; v < 4; ++v)
                if (!TAIL || v < valid || a.Lw >= 4) acc[v] = dst[v] + acc[v];
              if constexpr (TAIL) lanes_ordered();  // the last lane reads what its neighbour stores
            }
            store(row, dst, acc);
          }
        },
        [&](auto r, uint32_t rb, i4_t b, i4_t s, i4_t e) {
          constexpr int R = decltype(r)::value, S = U / R;
          if constexpr (G <= 64 / R) {
            int2 z[U];
            float x[U][4], acc[R][4] = {};
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int n = e[u / S] - s[u / S], k = u % S * NPP + g;
              z[u] = nz[(int)(s[u / S] - pb) + (k < n ? k : n - 1)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) load_e(x[u], z[u].x);
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (u % S * NPP + g < e[u / S] - s[u / S]) add(acc[u / S], x[u], z[u]);
            float o[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = groups_sum_of<R, G>(acc, v);
            const int k = value_of<R>(ln);
            uint32_t row = rb + (k == 0 ? b.x : b.y);
            if constexpr (R == 4) row = k < 2 ? row : rb + (k == 2 ? b.z : b.w);
            if (lane_in && (ln & (64 / R - 1)) < G) {
              float *dst = row_at(row) + col;
              if (row == crow) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                  if (!TAIL || v < valid || a.Lw >= 4) o[v] = dst[v] + o[v];
                if constexpr (TAIL) lanes_ordered();
              }
              store(row, dst, o);
            }
          }
        },
        [&](uint32_t row, uint32_t s, int n) {
          int2 z[U];
          float x[U][4], acc[4] = {0.f, 0.f, 0.f, 0.f};
          bool any[U];
#pragma unroll
          for (int u = 0; u < U; ++u) z[u] = nz[(int)(s - pb) + (u < n ? u : n - 1)];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            any[u] = u < 2 || __ballot(n > u) != 0;
            if (any[u]) load_e(x[u], z[u].x);
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (any[u] && u < n) add(acc, x[u], z[u]);
          if (lane_in) {
            float *dst = row_at(row) + col;
            if (row == crow) {
#pragma unroll
              for (int v = 0; v < 4; ++v)
                if (!TAIL || v < valid || a.Lw >= 4) acc[v] = dst[v] + acc[v];
            }
            lanes_ordered();  // groups that repeat a row, and the last lane, read what others store
            store(row, dst, acc);
          }
        });
  }

  // Zero rows (or partial rows) of the segments without a nonzero.
  __device__ __forceinline__ void zeros() {
    for (uint32_t rb = i0; rb <= rlast; rb += 64) {
      window(rb);
      uint64_t m = __ballot(rb + lane <= rlast && rb + lane != i1 && we <= ws);
      while (m) {
        const uint32_t row = rb + __builtin_ctzll(m);
        m &= m - 1;
        float *dst = row_at(row);
        for (int l = lane; l < a.Lw; l += 64) __builtin_nontemporal_store(0.f, dst + l);
      }
    }
  }

  __device__ __forceinline__ void run(const Part &s) {
    lane = threadIdx.x & 63;
    i0 = __builtin_amdgcn_readfirstlane((int)s.i0);
    p0 = __builtin_amdgcn_readfirstlane((int)s.p0);
    i1 = __builtin_amdgcn_readfirstlane((int)s.i1);
    p1 = __builtin_amdgcn_readfirstlane((int)s.p1);
    head = __builtin_amdgcn_readfirstlane((int)s.head);
    const int id = __builtin_amdgcn_readfirstlane((int)s.id);
    rlast = i1 < a.N ? i1 : i1 - 1;
    head_slot = a.carry + (int64_t)id * 2 * a.Lw;
    tail_slot = head_slot + a.Lw;
    wrb = kNoRow;
    if constexpr (MODE != kSddmm) zeros();
    uint32_t ib = i0, crow = kNoRow;
    for (uint32_t pb = p0; pb < p1;) {
      const uint32_t pe = p1 - pb < kBatch ? p1 : pb + kBatch;
      const int n = (int)(pe - pb);
      const int qk = (a.K + 3) >> 2;
      const bool whole = MODE == kSpmm || qk <= a.tk;  // one tile holds all of K
      int2 z[kBatch / 64];
#pragma unroll
      for (int t = 0; t < kBatch / 64; ++t) {
        const int k = t * 64 + lane;
        z[t] = int2{0, 0};
        if (k < n) {
          z[t].x = ld_stream(a.colidx + pb + k);
          if (whole) z[t].y = __builtin_bit_cast(int, ld_stream(a.vals + pb + k));
        }
      }
#pragma unroll
      for (int t = 0; t < kBatch / 64; ++t)
        if (t * 64 + lane < n) nz[t * 64 + lane] = z[t];
      lanes_ordered();
      // the first row with nonzeros from pe on, and whether it has some before
      uint32_t inext = ib, orow = kNoRow;
      if (pe < p1) {
        while (inext <= rlast) {
          window(inext);
          const uint64_t m = __ballot(inext + lane <= rlast && we > pe);
          if (m) {
            const int b = __builtin_ctzll(m);
            inext += b;
            if ((uint32_t)__builtin_amdgcn_readlane(ws, b) < pe) orow = inext;
            break;
          }
          inext += 64;
        }
      }
      if constexpr (MODE != kSpmm) {
        for (int q0 = 0; q0 < qk; q0 += a.tk) {
          const int nq = qk - q0 < a.tk ? qk - q0 : a.tk;
          if (nq <= 4) dots<4>(ib, pb, pe, q0, nq, whole);
          else if (nq <= 8) dots<8>(ib, pb, pe, q0, nq, whole);
          else if (nq <= 16) dots<16>(ib, pb, pe, q0, nq, whole);
          else if (nq <= 32) dots<32>(ib, pb, pe, q0, nq, whole);
          else dots<64>(ib, pb, pe, q0, nq, whole);
          lanes_ordered();
        }
        if (!whole || qk == 0 || MODE == kSddmm) {
          for (int t = lane; t < n; t += 64) {
            float y = __builtin_bit_cast(float, nz[t].y);
            if (qk == 0) y *= 0.f;  // K = 0: b times an empty sum
            else if (!whole) y *= ld_stream(a.vals + pb + t);
            if constexpr (MODE == kSddmm) a.out[pb + t] = y;
            else nz[t].y = __builtin_bit_cast(int, y);
          }
          lanes_ordered();
        }
      }
      if constexpr (MODE != kSddmm) {
        const int q4 = (a.Lw + 3) >> 2;
        for (int q0 = 0; q0 < q4; q0 += a.tl) {
          const int nq = q4 - q0 < a.tl ? q4 - q0 : a.tl;
          if (nq <= 4) rows<4>(ib, pb, pe, q0, nq, crow);
          else if (nq <= 8) rows<8>(ib, pb, pe, q0, nq, crow);
          else if (nq <= 16) rows<16>(ib, pb, pe, q0, nq, crow);
          else if (nq <= 32) rows<32>(ib, pb, pe, q0, nq, crow);
          else rows<64>(ib, pb, pe, q0, nq, crow);
        }
      }
      lanes_ordered();  // the next batch's copy, and what it adds to a row of A
      ib = inext;
      crow = orow;
      pb = pe;
    }
    if (MODE != kSddmm && s.last && i1 < a.N && p1 <= (uint32_t)a.rowptr[i1]) {  // an empty tail
      for (int l = lane; l < a.Lw; l += 64) tail_slot[l] = 0.f;
    }
    if (MODE != kSddmm && lane == 0) {
      int32_t *meta = a.meta + 2 * (int64_t)id;
      if (s.last) meta[0] = i1 < a.N ? (int)i1 : -1;
      if (s.first) meta[1] = s.head_row;
    }
  }
};

// Four gathers in flight per lane and six waves per SIMD; eight gathers need
// 120 registers and leave four.  SDDMM, with fewer registers, has seven: with six the
// 27-point stencils take 11% longer at K = 32 (114^3 635 -> 704 us), if 25% less at 64.
// The fused kernels keep 20 to 25 scalars in lanes of vector registers, those of ragged
// widths 55 to 65, which costs them 1 to 3%.
template <int MODE, bool TAIL, bool BIG>
__global__ __launch_bounds__(64) 
    __attribute__((amdgpu_waves_per_eu(MODE == kSddmm ? 7 : 6))) void walk_batch(WalkArgs a) {
  __shared__ int2 nonzeros[kBatch];
  const Part s = make_part(a);
  if (!s.active) return;
  BatchWalk<MODE, TAIL, BIG> w(a, nonzeros);
  w.run(s);
}

}  // namespace slnr

// Device code of the batch walk of the fused SDDMM->SpMM library for gfx950:
// the kernel for widths without a variant of their own, for operands off 16
// bytes, and for arrays of 4 GiB and more.
//
// A wave takes a merge-path slice (walker.hpp) in batches of kBatch nonzeros,
// whose columns it copies to LDS.  In one pass over the rows of the batch it
// forms the dot products, y = b * dot(C_i, D_j), beside the columns in LDS; in
// a second pass it adds y * E_j into the rows of A.  In both passes G lanes
// take four floats each of a gathered row, so 64 / G nonzeros of one row go
// side by side, and U such groups of gathers are issued before the first is
// used.  Lane count and column tile depend on the width alone, at run time:
// every width from 1 to 256 floats takes one tile, a wider one equal tiles.
//
// What bounds it is the fabric that the L2 misses go through: at 100003
// power-law rows of 25 nonzeros, K = 100, L = 47, 16M lines of 128 bytes are
// touched (6.5 per nonzero, as rows straddle lines) in 267 us, 60 lines a
// nanosecond, where plain streaming walks reach 58.  One nonzero at a time
// with one float per lane, which this kernel replaces, took 564 us; SpMM of
// 300007 rows of 20 nonzeros at L = 96: 843 -> 331 us; K = 259, L = 261 at
// 20011 rows of 11: 410 -> 113 us.
#pragma once

#include "walker.hpp"

namespace slnr {

// Nonzeros of a batch (8 bytes of LDS each).  512 leaves occupancy to the
// registers; with 1024 (measured) widths of 64 and 100 ran 2-11% slower.
constexpr int kBatch = 512;

typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u2_t __attribute__((ext_vector_type(2)));

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
  if constexpr (G <= 4) v += dpp<0x124>(v);  // row_ror:4
  if constexpr (G <= 8) v += dpp<0x128>(v);  // row_ror:8
  if constexpr (G <= 16) v = add_row16(v);
  if constexpr (G <= 32) v = add_half(v);
  return v;
}

// Floats col .. col+3 of row j; of a row too narrow for that (not `wide`) only
// the first `valid`.
template <bool TAIL, bool BIG>
__device__ __forceinline__ void ld_cols(float (&r)[4], const float *base, int j, int64_t stride,
                                        int col, bool wide, int valid) {
  const float *p;
  if constexpr (BIG) {
    p = base + (int64_t)j * stride + col;
  } else {
    const uint32_t off = __umul24((uint32_t)j, (uint32_t)stride * 4u) + (uint32_t)col * 4u;
    p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + off);
  }
  if (!TAIL || wide) {  // uniform
    const f4u_t x = *reinterpret_cast<const f4u_t *>(p);
    r[0] = x[0]; r[1] = x[1]; r[2] = x[2]; r[3] = x[3];
  } else {
    r[0] = r[1] = r[2] = r[3] = 0.f;
    if (valid > 0) r[0] = p[0];
    if (valid > 1) r[1] = p[1];
    if (valid > 2) r[2] = p[2];
  }
}

// TAIL: K or L is no multiple of 4.  BIG: 64-bit row offsets.
template <int MODE, bool TAIL, bool BIG>
struct BatchWalk {
  const WalkArgs &a;
  int2 *nz;
  int lane;
  int i0, p0, i1, p1;  // the slice
  bool head;
  int rlast;           // last row with a segment in the slice
  float *head_slot, *tail_slot;
  int wrb;             // rowptr window: row wrb + lane covers ws .. we of the slice
  int ws, we;

  __device__ __forceinline__ BatchWalk(const WalkArgs &a_, int2 *nz_) : a(a_), nz(nz_) {}

  __device__ __forceinline__ void window(int rb) {
    if (rb == wrb) return;
    wrb = rb;
    const int r = rb + lane;
    const bool in = r <= rlast;
    const int x = in ? a.rowptr[r] : 0, y = in ? a.rowptr[r + 1] : 0;
    ws = x > p0 ? x : p0;
    we = y < p1 ? y : p1;
    if (!in) ws = we = 0;
  }

  // f(row, s, e, cont, open) for every row with nonzeros s .. e-1 in the
  // batch [pb, pe); cont / open: it has nonzeros in an earlier batch of the
  // slice / does not end here.
  template <typename F>
  __device__ __forceinline__ void for_rows(int ib, int pb, int pe, F f) {
    for (int rb = ib;; rb += 64) {
      window(rb);
      const int vs = ws > pb ? ws : pb, ve = we < pe ? we : pe;
      uint64_t mask = __ballot(ve > vs);
      const bool more = rb + 63 < rlast && __builtin_amdgcn_readlane(we, 63) < pe;
      while (mask) {
        const int b = __builtin_ctzll(mask);
        mask &= mask - 1;
        const int row = rb + b;
        f(row, __builtin_amdgcn_readlane(vs, b), __builtin_amdgcn_readlane(ve, b),
          __builtin_amdgcn_readlane(ws, b) < pb,
          row == i1 || __builtin_amdgcn_readlane(we, b) > pe);
      }
      if (!more) return;
    }
  }

  // Partial dot products of the batch over floats [4 * q0, 4 * q0 + 4 * nq) of
  // the K floats: added to the y of every nonzero.
  template <int G>
  __device__ __forceinline__ void dots(int ib, int pb, int pe, int q0, int nq) {
    constexpr int NPP = 64 / G, U = 4;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // keeps the lane's indices out of the registers of other phases
    const int g = ln / G, q = ln & (G - 1);
    const int first = 4 * (q0 + q);
    const bool lane_in = q < nq;
    const int valid = a.K - first;
    // the last lane of a ragged width reads the last four floats and drops
    // those that the lane before it has
    const int col = TAIL && valid < 4 && a.K >= 4 ? a.K - 4 : first;
    const int drop = first - col;
    for_rows(ib, pb, pe, [&](int row, int s, int e, bool, bool) {
      float c[4] = {0.f, 0.f, 0.f, 0.f};
      if (lane_in) ld_cols<TAIL, true>(c, a.C, row, a.K, col, a.K >= 4, valid);
      for (int k = s; k < e; k += U * NPP) {
        const int n = e - k;
        int2 *zp = nz + (k - pb);
        int2 z[U];
        float x[U][4];
        auto finish = [&](int u, int idx) {
          float t = 0.f;
          if constexpr (TAIL) {
#pragma unroll
            for (int v = 0; v < 3; ++v) x[u][v] = v < drop ? 0.f : x[u][v];
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) t = fmaf(c[v], x[u][v], t);
          t = lanes_sum<G>(lane_in ? t : 0.f);
          if (q == 0) zp[idx].y = __builtin_bit_cast(int, __builtin_bit_cast(float, z[u].y) + t);
        };
        if (n >= U * NPP) {
#pragma unroll
          for (int u = 0; u < U; ++u) z[u] = zp[u * NPP + g];
          if (lane_in) {
#pragma unroll
            for (int u = 0; u < U; ++u) ld_cols<TAIL, BIG>(x[u], a.D, z[u].x, a.K, col, a.K >= 4, valid);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) finish(u, u * NPP + g);
        } else {  // groups past the row's end repeat its last nonzero
          auto at = [&](int u) { return u * NPP + g < n ? u * NPP + g : n - 1; };
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u * NPP < n) z[u] = zp[at(u)];
          if (lane_in) {
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (u * NPP < n) ld_cols<TAIL, BIG>(x[u], a.D, z[u].x, a.K, col, a.K >= 4, valid);
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u * NPP < n) finish(u, at(u));
        }
      }
    });
  }

  // Columns l0 + [4 * q0, 4 * q0 + 4 * nq) of the rows of the batch.
  template <int G>
  __device__ __forceinline__ void rows(int ib, int pb, int pe, int q0, int nq) {
    constexpr int NPP = 64 / G, U = 4;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // keeps the lane's indices out of the registers of other phases
    const int g = ln / G, q = ln & (G - 1);
    const int first = 4 * (q0 + q);
    const bool lane_in = q < nq;
    const int valid = a.Lw - first;
    // the last lane of a ragged width takes the last four columns: it forms
    // and stores the same values as its neighbour where they overlap
    const int col = TAIL && valid < 4 && a.Lw >= 4 ? a.Lw - 4 : first;
    for_rows(ib, pb, pe, [&](int row, int s, int e, bool cont, bool open) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      for (int k = s; k < e; k += U * NPP) {
        const int n = e - k;
        const int2 *zp = nz + (k - pb);
        int2 z[U];
        float x[U][4];
        auto add = [&](int u) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            acc[v] = fmaf(__builtin_bit_cast(float, z[u].y), x[u][v], acc[v]);
        };
        if (n >= U * NPP) {
#pragma unroll
          for (int u = 0; u < U; ++u) z[u] = zp[u * NPP + g];
          if (lane_in) {
#pragma unroll
            for (int u = 0; u < U; ++u) ld_cols<TAIL, BIG>(x[u], a.E, z[u].x, a.L, a.l0 + col, a.Lw >= 4, valid);
#pragma unroll
            for (int u = 0; u < U; ++u) add(u);
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u * NPP < n) z[u] = zp[u * NPP + g < n ? u * NPP + g : n - 1];
          if (lane_in) {
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (u * NPP < n) ld_cols<TAIL, BIG>(x[u], a.E, z[u].x, a.L, a.l0 + col, a.Lw >= 4, valid);
#pragma unroll
            for (int u = 0; u < U; ++u) {
              if ((u + 1) * NPP <= n) add(u);
              else if (u * NPP < n && u * NPP + g < n) add(u);
            }
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = groups_sum<G>(acc[v]);
      if (lane_in && g == 0) {
        float *dst = open ? tail_slot + col
                          : row == i0 && head ? head_slot + col
                                              : a.out + (int64_t)row * a.L + a.l0 + col;
        if (!TAIL || a.Lw >= 4) {
          if (cont) {
            const f4u_t o = *reinterpret_cast<const f4u_t *>(tail_slot + col);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] = o[v] + acc[v];
          }
          f4u_t o;
          o[0] = acc[0]; o[1] = acc[1]; o[2] = acc[2]; o[3] = acc[3];
          *reinterpret_cast<f4u_t *>(dst) = o;
        } else {
#pragma unroll
          for (int v = 0; v < 3; ++v)
            if (v < valid) dst[v] = (cont ? tail_slot[col + v] : 0.f) + acc[v];
        }
      }
    });
  }

  // Zero rows (or partial rows) of the segments without a nonzero.
  __device__ __forceinline__ void zeros() {
    for (int rb = i0; rb <= rlast; rb += 64) {
      window(rb);
      uint64_t m = __ballot(rb + lane <= rlast && rb + lane != i1 && we <= ws);
      while (m) {
        const int row = rb + __builtin_ctzll(m);
        m &= m - 1;
        float *dst = row == i0 && head ? head_slot : a.out + (int64_t)row * a.L + a.l0;
        for (int l = lane; l < a.Lw; l += 64) __builtin_nontemporal_store(0.f, dst + l);
      }
    }
  }

  __device__ __forceinline__ void run(const Slice &s) {
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
    wrb = -1;
    if constexpr (MODE != kSddmm) zeros();
    int ib = i0;
    for (int pb = p0; pb < p1;) {
      const int pe = p1 - pb < kBatch ? p1 : pb + kBatch;
      const int n = pe - pb;
      for (int t = lane; t < n; t += 64) {
        int2 z;
        z.x = ld_stream(a.colidx + pb + t);
        z.y = MODE == kSpmm ? __builtin_bit_cast(int, ld_stream(a.vals + pb + t)) : 0;
        nz[t] = z;
      }
      if constexpr (MODE != kSpmm) {
        const int q4 = (a.K + 3) >> 2;
        for (int q0 = 0; q0 < q4; q0 += a.tk) {
          const int nq = q4 - q0 < a.tk ? q4 - q0 : a.tk;
          if (nq <= 4) dots<4>(ib, pb, pe, q0, nq);
          else if (nq <= 8) dots<8>(ib, pb, pe, q0, nq);
          else if (nq <= 16) dots<16>(ib, pb, pe, q0, nq);
          else if (nq <= 32) dots<32>(ib, pb, pe, q0, nq);
          else dots<64>(ib, pb, pe, q0, nq);
        }
        for (int t = lane; t < n; t += 64) {
          const float y = ld_stream(a.vals + pb + t) * __builtin_bit_cast(float, nz[t].y);
          if constexpr (MODE == kSddmm) a.out[pb + t] = y;
          else nz[t].y = __builtin_bit_cast(int, y);
        }
      }
      if constexpr (MODE != kSddmm) {
        const int q4 = (a.Lw + 3) >> 2;
        for (int q0 = 0; q0 < q4; q0 += a.tl) {
          const int nq = q4 - q0 < a.tl ? q4 - q0 : a.tl;
          if (nq <= 4) rows<4>(ib, pb, pe, q0, nq);
          else if (nq <= 8) rows<8>(ib, pb, pe, q0, nq);
          else if (nq <= 16) rows<16>(ib, pb, pe, q0, nq);
          else if (nq <= 32) rows<32>(ib, pb, pe, q0, nq);
          else rows<64>(ib, pb, pe, q0, nq);
        }
      }
      // first row with nonzeros from pe on
      if (pe < p1) {
        while (ib <= rlast) {
          window(ib);
          const uint64_t m = __ballot(ib + lane <= rlast && we > pe);
          if (m) {
            ib += __builtin_ctzll(m);
            break;
          }
          ib += 64;
        }
      }
      pb = pe;
    }
    // A tail segment without a nonzero: its slot may hold a row carried from
    // one batch to the next, so it is cleared last.
    if (MODE != kSddmm && i1 < a.N && p1 <= a.rowptr[i1]) {
      for (int l = lane; l < a.Lw; l += 64) tail_slot[l] = 0.f;
    }
    if (MODE != kSddmm && lane == 0) {
      int32_t *meta = a.meta + 2 * (int64_t)id;
      meta[0] = i1 < a.N ? i1 : -1;
      meta[1] = head ? i0 : -1;
    }
  }
};

// Four gathers in flight per lane and six waves per SIMD; eight gathers need
// 120 registers and leave four.
template <int MODE, bool TAIL, bool BIG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) void walk_batch(WalkArgs a) {
  __shared__ int2 nonzeros[kBatch];
  const Slice s = make_slice<64>(a);
  if (!s.active) return;
  BatchWalk<MODE, TAIL, BIG> w(a, nonzeros);
  w.run(s);
}

}  // namespace slnr

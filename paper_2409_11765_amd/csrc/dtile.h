// Float64 products in which every wave of a workgroup computes the whole tile
// over its part of k.
#pragma once

#include <hip/hip_runtime.h>

namespace cmx {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// ---- products.  A workgroup computes a square tile of MB x MB MFMA blocks
// (16 x 16); every one of its NW waves computes the whole tile over its own
// part of k, and the partial sums meet in LDS.  v_mfma_f64_16x16x4 takes 64
// cycles for 2 x 64 operand values, so a wave that holds the whole tile needs
// few bytes per cycle and reads its operands straight from global memory into
// the fragment registers: no LDS and no barrier in the k-loop, two chunks of 16
// k in flight.  Both operands are read along k with 16-byte loads: lane (i = l
// & 15, g = l >> 4) holds k = 16 c + 8 h + 2 g + s of row i (h, s = 0, 1), so
// the four lanes of a row read 64 consecutive bytes, and instruction (h, s) of
// a chunk multiplies those k of all four g.  TA = false reads A(m, k) along m
// instead.  The operands change roles in the instruction, so that 16
// consecutive lanes of a result are 16 consecutive rows.
// MB = 3, NW = 4: two workgroups per CU; at n = 1000 a whole product is 441
// tiles and two lower triangles are 462, both just under the 512 the chip
// holds (41 us for a whole product; with 64 x 64 tiles of 32 x 32 per wave, 256
// and 272 tiles, 50 and 120 us).  The smaller tiles give more workgroups and a
// shorter k-loop each: at n = 200 a product takes 4.1 us with MB = 1, NW = 4
// against 7.4-8.5 with MB = 2, NW = 8, at n = 333 7.5-9.0 against 9.9-12.2.
template <int MB_, int NW_>
struct Tile {
  static constexpr int MB = MB_, NW = NW_;
  static constexpr int T = 16 * MB;
  static constexpr int THREADS = 64 * NW;
  static constexpr int PER = T * T / THREADS;  // elements per thread
  static constexpr int PS = T + 1;             // LDS column stride
  static constexpr int LDS = NW * T * PS;      // doubles
  static_assert(PER * THREADS == T * T, "elements must split evenly");

  struct Frag {
    double a[MB][4], b[MB][4];
  };

  // the tile at (m0, n0) of op(A) B over kc chunks of 16 k, partial sums in
  // lds; rows and columns are clamped to rmax and cmax (their results are
  // ignored).  CLAMP: A's k is clamped to kmax; with TA that is a multiple of 4
  // past which any stored value is read, for B's zero rows; else it is the
  // number of k there are, and B's past it, whatever they hold, count as zero.
  // TB (with CLAMP, without TA): B(k, n) is read along n.
  // Nothing is computed, and false returned, unless go (uniform; tested when the
  // first loads are under way).
  template <bool TA, bool CLAMP, bool TB = false>
  __device__ static bool product(double* lds, const double* __restrict__ A, int lda, const double* __restrict__ B,
                                 int ldb, int kc, int m0, int n0, int rmax, int cmax, int kmax, bool go) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const int c0 = wave * kc / NW, c1 = (wave + 1) * kc / NW;
    const double *pa[MB], *pb[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = min(m0 + 16 * i + li, rmax - 1), col = min(n0 + 16 * i + li, cmax - 1);
      pa[i] = TA ? A + static_cast<int64_t>(row) * lda + 2 * lg : A + static_cast<int64_t>(2 * lg) * lda + row;
      pb[i] = TB ? B + static_cast<int64_t>(2 * lg) * ldb + col : B + static_cast<int64_t>(col) * ldb + 2 * lg;
    }
    doublex4 acc[MB][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < MB; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    auto load = [&](Frag& f, int c) {
      const int k = 16 * min(c, c1 - 1);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if constexpr (TA) {
            int o = k + 8 * h;
            if constexpr (CLAMP) o = o + 2 * lg < kmax ? o : -2 * lg;
            const double2 x = *reinterpret_cast<const double2*>(pa[i] + o);
            f.a[i][2 * h] = x.x;
            f.a[i][2 * h + 1] = x.y;
          } else {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              int o = k + 8 * h + s;
              if constexpr (CLAMP) o = min(o, kmax - 1 - 2 * lg);
              f.a[i][2 * h + s] = pa[i][static_cast<int64_t>(o) * lda];
            }
          }
          if constexpr (TB) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              const int o = k + 8 * h + s, left = kmax - 2 * lg - o;
              const double y = pb[i][static_cast<int64_t>(left > 0 ? o : -2 * lg) * ldb];
              f.b[i][2 * h + s] = left > 0 ? y : 0.0;
            }
          } else if constexpr (CLAMP && !TA) {
            // (a pair's second element may be the first one of the padding)
            const int o = k + 8 * h, left = kmax - 2 * lg - o;
            const double2 y = *reinterpret_cast<const double2*>(pb[i] + (left > 0 ? o : -2 * lg));
            f.b[i][2 * h] = left > 0 ? y.x : 0.0;
            f.b[i][2 * h + 1] = left > 1 ? y.y : 0.0;
          } else {
            const double2 y = *reinterpret_cast<const double2*>(pb[i] + k + 8 * h);
            f.b[i][2 * h] = y.x;
            f.b[i][2 * h + 1] = y.y;
          }
        }
      }
    };
    auto compute = [&](const Frag& f) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < MB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.b[j][s], f.a[i][s], acc[i][j], 0, 0, 0);
    };
    if (c0 < c1) {
      Frag f0, f1;
      load(f0, c0);
      load(f1, c0 + 1);
      if (!go) return false;
      // (no branch inside: the waits then count the loads in flight exactly)
      int c = c0;
      for (; c + 1 < c1; c += 2) {
        compute(f0);
        load(f0, c + 2);
        __builtin_amdgcn_sched_barrier(0);
        compute(f1);
        load(f1, c + 3);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (c < c1) compute(f0);
    } else if (!go) {
      return false;
    }
    double* p = lds + wave * T * PS;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[(16 * j + lg + 4 * r) * PS + 16 * i + li] = acc[i][j][r];
    __syncthreads();
    return true;
  }
  // element (r, c) of the tile: the waves' sums in order
  __device__ static double get(const double* lds, int r, int c) {
    const double* p = lds + c * PS + r;
    double v = p[0];
#pragma unroll
    for (int g = 1; g < NW; ++g) v += p[g * T * PS];
    return v;
  }
  // the tile's transpose to out (rows n0.., columns m0..): thread values v[e]
  // of the elements (r, c) with r + T c = threadIdx.x + THREADS e, through LDS
  __device__ static void store_mirror(double* lds, const double (&v)[PER], double* __restrict__ out, int N, int m0,
                                      int n0) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int idx = threadIdx.x + THREADS * e;
      lds[(idx % T) * PS + idx / T] = v[e];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int idx = threadIdx.x + THREADS * e, r = idx % T, c = idx / T;  // row n0 + r, column m0 + c
      if (n0 + r < N && m0 + c < N) out[static_cast<int64_t>(m0 + c) * N + n0 + r] = lds[c * PS + r];
    }
  }
};

// workgroup b of a launch of `total` to its tile number: workgroups go to the
// 8 XCDs in turn, and each XCD gets a contiguous run of tiles (its L2 then
// holds the operands of that run)
__device__ __forceinline__ int xcd_order(int b, int total) {
  const int per = total / 8, extra = total % 8, x = b % 8, i = b / 8;
  return x * per + min(x, extra) + i;
}

}  // namespace cmx

// The general kernel: contractions over any index pairs (IndexMap, desc.hpp) in
// FP64 and FP32, as the GEMM C(m, n) = sum_k A(m, k) B(k, n) whose element
// offsets are sums of a row's and a column's: a_row[m] + a_k[k], b_k[k] +
// b_col[n], c_row[m] + c_col[n].
#pragma once
#include "hec.hpp"

namespace cdag {

// Element offset of a mixed-radix index x (nd digits in radix n, most
// significant first) with per-digit strides st.
__device__ __forceinline__ int64_t digit_offset(uint32_t x, int nd, uint32_t n, const int64_t* st) {
  int64_t off = 0;
#pragma unroll
  for (int d = 2; d >= 0; --d) {
    if (d < nd) {
      off += (int64_t)(x % n) * st[d];
      x /= n;
    }
  }
  return off;
}

// One work item is a 32 x 32 output tile (four waves of one 16 x 16 block each,
// three real products per complex one, as hec_mfma on that tile) with the whole
// K, in k-slices of 32 through one LDS stage and a register prefetch.
//
// The offsets of the tile's rows and columns and of up to KT k are worked out
// once into LDS, so that a load is one address sum: with the digits divided out
// for every element the divisions, not the loads or the products, were the
// bound.  The threads of a load or a store run along the axis whose digit has
// stride 1 (the host puts it last in its index, index_map), so that a wave
// reads and writes whole runs; the output tile is turned through LDS for that.
// Where neither index of an operand ends in its unit-stride axis (it is an
// earlier digit of a summed or shared index) the loads stay scattered and lean
// on the caches.
// Measured (FP64, N = 20, Nt 4, two launches of 30 graphs' contractions):
// 0.57 -> 0.14 ms.
template <typename T>
__global__ void __launch_bounds__(256) hec_general(char* __restrict__ arena, const HecDesc* __restrict__ descs,
                                                   Span n_desc, int64_t n_items, const HcaDesc*, Span, int64_t) {
  typedef typename Mfma<T>::V V;
  constexpr int B = 32, BK = 32, PAD = BK + 1, KT = 256;
  constexpr int E = 2 * B * BK / 256;   // elements of A, and of B, per thread and slice
  constexpr int OPER = 2 * B * PAD;
  __shared__ __attribute__((aligned(16))) T smem[2 * OPER];
  __shared__ int64_t a_row[B], b_col[B], c_row[B], c_col[B], a_k[KT], b_k[KT];
  T (&As)[2][B][PAD] = *reinterpret_cast<T (*)[2][B][PAD]>(smem);          // [plane][m][k]
  T (&Bs)[2][BK][PAD] = *reinterpret_cast<T (*)[2][BK][PAD]>(smem + OPER);  // [plane][k][n]
  T (&Cs)[2][B][PAD] = *reinterpret_cast<T (*)[2][B][PAD]>(smem);          // [plane][m][n]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, li = lane & 15, lk = lane >> 4;

  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    const ItemView<T> o = view_item<T, B, B>(arena, descs, n_desc, item);
    const IndexMap& mp = *o.map;
    const int64_t a_plane = (int64_t)o.M * o.K, b_plane = (int64_t)o.K * o.N, c_plane = (int64_t)o.M * o.N;
    const bool a_by_m = mp.dm > 0 && mp.a_m[mp.dm - 1] == 1, b_by_n = mp.dn > 0 && mp.b_n[mp.dn - 1] == 1;
    const bool c_by_m = mp.dm > 0 && mp.c_m[mp.dm - 1] == 1;
    // rows, columns and k past the end take the last one's offsets
    auto fill_k = [&](int k0) {
      const uint32_t k = min(k0 + tid, o.K - 1);
      a_k[tid] = digit_offset(k, mp.dk, mp.n, mp.a_k);
      b_k[tid] = digit_offset(k, mp.dk, mp.n, mp.b_k);
    };
    static_assert(KT == 256, "one k per thread");
    __syncthreads();   // the previous item's tile has been stored
    if (tid < B) {
      const uint32_t m = min(o.m0 + tid, o.M - 1);
      a_row[tid] = digit_offset(m, mp.dm, mp.n, mp.a_m);
      c_row[tid] = digit_offset(m, mp.dm, mp.n, mp.c_m);
    } else if (tid >= 64 && tid < 64 + B) {
      const uint32_t n = min(o.n0 + tid - 64, o.N - 1);
      b_col[tid - 64] = digit_offset(n, mp.dn, mp.n, mp.b_n);
      c_col[tid - 64] = digit_offset(n, mp.dn, mp.n, mp.c_n);
    }
    fill_k(0);
    __syncthreads();

    T ra[E], rb[E];
    // element e of the slice: plane e / 1024, then (row, k) with the fast index
    // along the unit-stride axis
    auto gload = [&](int k0) {
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int e = tid + 256 * q, p = e >> 10, slow = (e >> 5) & 31, fast = e & 31;
        const int r = a_by_m ? fast : slow, k = a_by_m ? slow : fast;
        ra[q] = o.A[p * a_plane + a_row[r] + a_k[(k0 + k) % KT]];
      }
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int e = tid + 256 * q, p = e >> 10, slow = (e >> 5) & 31, fast = e & 31;
        const int c = b_by_n ? fast : slow, k = b_by_n ? slow : fast;
        rb[q] = o.B[p * b_plane + b_k[(k0 + k) % KT] + b_col[c]];
      }
    };
    V p1 = V{0, 0, 0, 0}, p2 = V{0, 0, 0, 0}, p3 = V{0, 0, 0, 0};
    gload(0);
    for (int k0 = 0; k0 < o.K; k0 += BK) {
      const int left = o.K - k0;
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const int e = tid + 256 * q, p = e >> 10, slow = (e >> 5) & 31, fast = e & 31;
        const int ka = a_by_m ? slow : fast, kb = b_by_n ? slow : fast;
        As[p][a_by_m ? fast : slow][ka] = ka < left ? ra[q] : T(0);
        Bs[p][kb][b_by_n ? fast : slow] = kb < left ? rb[q] : T(0);
      }
      __syncthreads();
      if (left > BK) {
        if ((k0 + BK) % KT == 0) {   // every thread's loads of this table are done
          fill_k(k0 + BK);
          __syncthreads();
        }
        gload(k0 + BK);
      }
      const int n4 = min(BK / 4, (left + 3) / 4);
      auto step = [&](int k4) {
        const int kk = 4 * k4 + lk;
        const T ar = As[0][wm * 16 + li][kk], ai = As[1][wm * 16 + li][kk];
        const T br = Bs[0][kk][wn * 16 + li], bi = Bs[1][kk][wn * 16 + li];
        p1 = Mfma<T>::mma(ar, br, p1);
        p2 = Mfma<T>::mma(ai, bi, p2);
        p3 = Mfma<T>::mma(ar + ai, br + bi, p3);
      };
      if (n4 == BK / 4) {
#pragma unroll
        for (int k4 = 0; k4 < BK / 4; ++k4) step(k4);
      } else {
#pragma unroll 1
        for (int k4 = 0; k4 < n4; ++k4) step(k4);
      }
      __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = wm * 16 + Mfma<T>::row(lk, v), c = wn * 16 + li;
      Cs[0][r][c] = p1[v] - p2[v];
      Cs[1][r][c] = p3[v] - (p1[v] + p2[v]);
    }
    __syncthreads();
    T* C = reinterpret_cast<T*>(arena + o.h->c_off) + (int64_t)o.t * 2 * c_plane;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int e = tid + 256 * q, p = e >> 10, slow = (e >> 5) & 31, fast = e & 31;
      const int r = c_by_m ? fast : slow, c = c_by_m ? slow : fast;
      if (o.m0 + r < o.M && o.n0 + c < o.N) C[p * c_plane + c_row[r] + c_col[c]] = Cs[p][r][c];
    }
  }
}

}  // namespace cdag

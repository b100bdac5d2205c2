// Split fp32 products (split3.h) with rows that are contiguous in the
// contraction index, or k-major, on either side: the large-vocabulary head's
// logits and dL/dh, and dX.
#include <algorithm>

#include "lstm_dev.h"
#include "split3.h"

namespace cavs {
namespace {

// Operand loaders: thread t of 128 fetches 32 values of the 128-row, 32-deep
// chunk at k0 (zeros past the operand or past kend) and writes them, split,
// to LDS rows 32 j + i (tile rows 4 i + j).
//
// Rows contiguous in k: four adjacent rows, eight k each.
struct X3Rows {
  const float* base;
  long long ld;
  int rows;
  struct State {
    const float* p[4];
    int q, i;
  };
  __device__ void init(const Net&, State& s, int t, int r0) const {
    s.q = t & 3;
    s.i = t >> 2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 4 * s.i + j;
      s.p[j] = r < rows ? base + (size_t)r * ld + 8 * s.q : nullptr;
    }
  }
  __device__ static void load(const Net& n, const State& s, int k0, int kend, float4 (&v)[8]) {
    const int k = k0 + 8 * s.q;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)   // K is a multiple of 4
        v[2 * j + h] = ldg4(s.p[j] && k + 4 * h < kend ? s.p[j] + k0 + 4 * h : n.zrow);
  }
  __device__ static void store(char* lds, const State& s, const float4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float x[8] = {v[2 * j].x,     v[2 * j].y,     v[2 * j].z,     v[2 * j].w,
                          v[2 * j + 1].x, v[2 * j + 1].y, v[2 * j + 1].z, v[2 * j + 1].w};
      x3_store(lds, 32 * j + s.i, s.q, x);
    }
  }
};

// k-major: eight k rows, four adjacent columns.
struct X3Cols {
  const float* base;
  long long ld;
  int cols;
  struct State {
    const float* p;
    long long ld;
    int q, i;
  };
  __device__ void init(const Net&, State& s, int t, int r0) const {
    s.q = t >> 5;
    s.i = t & 31;
    const int c = r0 + 4 * s.i;
    s.ld = ld;
    s.p = c < cols ? base + c : nullptr;
  }
  __device__ static void load(const Net& n, const State& s, int k0, int kend, float4 (&v)[8]) {
    const int k = k0 + 8 * s.q;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ldg4(s.p && k + e < kend ? s.p + (k + e) * s.ld : n.zrow);
  }
  __device__ static void store(char* lds, const State& s, const float4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = j == 0 ? v[e].x : j == 1 ? v[e].y : j == 2 ? v[e].z : v[e].w;
      x3_store(lds, 32 * j + s.i, s.q, x);
    }
  }
};

// out[z][m][c] = sum over k in [z kchunk, (z + 1) kchunk) of A B^T; the tile
// and its pipeline as in k_x3_tn (lazy.hip).  Items: row tiles, then column
// tiles, then splits, a contiguous eighth to each XCD.
// WGS workgroups share a CU: three where their registers fit (168 each).
template <class LA, class LB, int WGS>
__global__ void __launch_bounds__(256, WGS) k_x3_gemm(Net n, LA la, LB lb, int M, int Nc, int K,
                                                    int kchunk, int items, float* out,
                                                    long long ldo) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kX3Bytes];
  const int item = xcd_item(blockIdx.x, items);
  if (item < 0) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wm = w & 1, wn = w >> 1;
  const int ty = cdiv_dev(M, kX3Tile), tx = cdiv_dev(Nc, kX3Tile), z = item / (tx * ty);
  const int m0 = item % ty * kX3Tile, n0 = item / ty % tx * kX3Tile;
  const int klo = z * kchunk, khi = min(K, klo + kchunk);
  const bool bside = __builtin_amdgcn_readfirstlane(tid >> 7) != 0;
  typename LA::State sa{};
  typename LB::State sb{};
  if (bside) lb.init(n, sb, tid & 127, n0);
  else la.init(n, sa, tid & 127, m0);
  v4f acc[4][4];
  zero_acc(acc);
  float4 v[8];
  auto load = [&](int k0) {
    if (bside) LB::load(n, sb, k0, khi, v);
    else LA::load(n, sa, k0, khi, v);
  };
  load(klo);
  for (int k0 = klo; k0 < khi; k0 += kBK) {
    if (k0 > klo) __syncthreads();   // the previous chunk's fragments are read
    if (bside) LB::store(lds + kX3Bytes, sb, v);
    else LA::store(lds, sa, v);
    __syncthreads();
    if (k0 + kBK < khi) load(k0 + kBK);
    __builtin_amdgcn_sched_barrier(0);   // the next chunk's loads go out before these products
    x3_mma(lds, lds + kX3Bytes, wm, wn, acc);
  }
  float* o = out + (size_t)z * M * Nc;
  const int nc = n0 + 64 * wn + 4 * r;
  if (nc >= Nc) return;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + 64 * wm + 16 * g + 4 * e + j;
      if (m < M)
        st4(o + (size_t)m * ldo + nc,
            make_float4(acc[j][0][e], acc[j][1][e], acc[j][2][e], acc[j][3][e]));
    }
}

}  // namespace

// Z[V, C] = h W_s: W_s as it is ([H, C], k-major).  2275 x 10 000 x 512:
// 233 us on fp32 instructions (and 16 us of transposing W_s) -> 135 us.
void lm_logits(const Net& n, hipStream_t s) {
  const int items = cdiv(n.C, kX3Tile) * cdiv(n.V, kX3Tile);
  CAVS_LAUNCH("k_x3_gemm<lm_logits>", (k_x3_gemm<X3Rows, X3Cols, 3>), dim3(xcd_grid(items)), dim3(256),
              0, s, n, X3Rows{n.Hs, n.H, n.V}, X3Cols{n.Ws, n.C, n.C}, n.V, n.C, n.H, n.H, items,
              n.dZ, (long long)n.C);
}

// dL/dh[V, H] = dZ W_s^T: a long contraction (C) over few tiles, so it is
// split until the grid is one round of 512 workgroups (scratch permitting)
// and the parts are added in order.  2275 x 512 x 10 000: 529 us (unsplit,
// 288 workgroups) -> 125 us and 8 us of adding.
void lm_dh(const Net& n, float* part, size_t part_floats, hipStream_t s) {
  const int tiles = cdiv(n.H, kX3Tile) * cdiv(n.V, kX3Tile), nch = cdiv(n.C, kBK);
  const size_t out = (size_t)n.V * n.H;
  int S = std::max(1, std::min({512 / tiles, nch / 4, (int)std::min<size_t>(part_floats / out, 64)}));
  const int kchunk = cdiv(nch, S) * kBK;
  S = cdiv(n.C, kchunk);
  CAVS_LAUNCH("k_x3_gemm<lm_dh>", (k_x3_gemm<X3Rows, X3Rows, 2>), dim3(xcd_grid(tiles * S)), dim3(256),
              0, s, n, X3Rows{n.dZ, n.C, n.V}, X3Rows{n.Ws, n.C, n.H}, n.V, n.H, n.C, kchunk,
              tiles * S, S > 1 ? part : n.dHL, (long long)n.H);
  if (S == 1) return;
  SplitJobs jobs;
  jobs.j[jobs.n++] = SplitJob{part, n.dHL, S, n.V, n.H, n.H, 0, 1 << 30, 0};
  reduce_split_jobs(jobs, s);
}

}  // namespace cavs

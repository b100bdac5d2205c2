// Products on the bf16 matrix cores with operands split (fp32) or rounded
// (bf16) on their way to LDS (split3.h), rows contiguous in the contraction
// index or k-major on either side: the large-vocabulary head's logits and
// dL/dh, the pull product (bf16, and fp32 over many rows), bf16 dX of many rows.
#include <algorithm>
#include <type_traits>

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
  __device__ void load(const Net& n, const State& s, int k0, int kend, float4 (&v)[8]) const {
    const int k = k0 + 8 * s.q;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)   // K is a multiple of 4
        v[2 * j + h] = ldg4(s.p[j] && k + 4 * h < kend ? s.p[j] + k0 + 4 * h : n.zrow);
  }
  template <int PARTS>
  __device__ static void store(char* lds, const State& s, const float4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float x[8] = {v[2 * j].x,     v[2 * j].y,     v[2 * j].z,     v[2 * j].w,
                          v[2 * j + 1].x, v[2 * j + 1].y, v[2 * j + 1].z, v[2 * j + 1].w};
      x3_store<PARTS>(lds, 32 * j + s.i, s.q, x);
    }
  }
};

// The same over the x rows of pulling positions (pull product).
struct X3Pulled : X3Rows {
  __device__ void init(const Net& n, State& s, int t, int r0) const {
    s.q = t & 3;
    s.i = t >> 2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 4 * s.i + j;
      s.p[j] = r < rows ? n.X + (size_t)n.pull_pos[n.pull_list[r]] * n.D + 8 * s.q : nullptr;
    }
  }
};

// Rows of W_x^T, LDS block j the gate block j of units r0 / 4 ..: a lane of
// the product then holds every gate of its unit.
struct X3Gates : X3Rows {
  __device__ void init(const Net& n, State& s, int t, int r0) const {
    s.q = t & 3;
    s.i = t >> 2;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      s.p[j] = n.WxT + ((size_t)j * n.H + r0 / 4 + s.i) * n.D + 8 * s.q;
  }
};

// bf16 dX: dA rows of pulling positions against rows of W_x, k over the gate
// columns: i|o|u (the f block skipped), or with_f all of them, the slots'
// forget blocks summed (the sum is what is rounded).
struct X3DxA : X3Rows {
  int with_f;
  __device__ void init(const Net& n, State& s, int t, int r0) const {
    s.q = t & 3;
    s.i = t >> 2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 4 * s.i + j;
      s.p[j] = r < rows ? n.dA + (size_t)n.pull_list[r] * n.GW + 8 * s.q : nullptr;
    }
  }
  __device__ void load(const Net& n, const State& s, int k0, int, float4 (&v)[8]) const {
    const int H = n.H, col = with_f || k0 < H ? k0 : k0 + H;
    const bool sum = col >= H && col < 2 * H;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v[2 * j + h] = ldg4(s.p[j] ? s.p[j] + col + 4 * h : n.zrow);
        if (sum)
          for (int k = 1; k < n.N; ++k)
            v[2 * j + h] = add4(v[2 * j + h], ldg4(s.p[j] ? s.p[j] + (2 + k) * H + col + 4 * h : n.zrow));
      }
  }
};
struct X3DxB : X3Rows {
  int with_f;
  __device__ void load(const Net& n, const State& s, int k0, int, float4 (&v)[8]) const {
    const int H = n.H, col = with_f || k0 < H ? k0 : k0 + H;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[2 * j + h] = ldg4(s.p[j] ? s.p[j] + col + 4 * h : n.zrow);
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
  __device__ void load(const Net& n, const State& s, int k0, int kend, float4 (&v)[8]) const {
    const int k = k0 + 8 * s.q;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ldg4(s.p && k + e < kend ? s.p + (k + e) * s.ld : n.zrow);
  }
  template <int PARTS>
  __device__ static void store(char* lds, const State& s, const float4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = j == 0 ? v[e].x : j == 1 ? v[e].y : j == 2 ? v[e].z : v[e].w;
      x3_store<PARTS>(lds, 32 * j + s.i, s.q, x);
    }
  }
};

// The blocks of X3Gates from W_x as it is (bf16): four units of one gate block.
// Most bf16 passes then transpose nothing, and the large ones stage faster: 10 to
// 448 pulled rows, D = 100, transpose and pull 13.3 to 18 us -> 8.5 to 11; 21 004,
// D = 300, H = 1024, 10 + 265 -> 7 (U alone) + 248; 18 901 at 512, inference, 5 + 99
// -> 5 + 88.
struct X3GatesK : X3Cols {
  __device__ void init(const Net& n, State& s, int t, int r0) const {
    const int i = t & 31, j = i >> 3, c = 4 * (i & 7);
    s.q = t >> 5;
    s.i = 32 * j + c;
    s.ld = 4LL * n.H;
    s.p = n.Wx + (size_t)j * n.H + r0 / 4 + c;
  }
  template <int PARTS>
  __device__ static void store(char* lds, const State& s, const float4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = j == 0 ? v[e].x : j == 1 ? v[e].y : j == 2 ? v[e].z : v[e].w;
      x3_store<PARTS>(lds, s.i + j, s.q, x);
    }
  }
};

// What a workgroup does with its 128 x 128 block: lane (r, g) of wavefront
// (wm, wn) holds rows 64 wm + 16 g + 4 e + j, columns 64 wn + 4 r .. + 3.
// Plain: out[z][m][c] (one block per split z of the contraction).
struct X3Out {
  float* out;
  long long ld;
  int rows, cols;
  __device__ void operator()(const Net&, int z, int m0, int n0, int wm, int wn, int g, int r,
                             const v4f (&acc)[4][4]) const {
    float* o = out + (size_t)z * rows * cols;
    const int nc = n0 + 64 * wn + 4 * r;
    if (nc >= cols) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 64 * wm + 16 * g + 4 * e + j;
        if (m < rows)
          st4(o + (size_t)m * ld + nc,
              make_float4(acc[j][0][e], acc[j][1][e], acc[j][2][e], acc[j][3][e]));
      }
  }
};
// dX rows of the pulled inputs.
struct X3DxOut {
  float* dX;
  int rows;
  __device__ void operator()(const Net& n, int, int m0, int n0, int wm, int wn, int g, int r,
                             const v4f (&acc)[4][4]) const {
    const int d = n0 + 64 * wn + 4 * r;
    if (d >= n.D) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 64 * wm + 16 * g + 4 * e + j;
        if (m < rows)
          st4(dX + (size_t)n.pull_pos[n.pull_list[m]] * n.D + d,
              make_float4(acc[j][0][e], acc[j][1][e], acc[j][2][e], acc[j][3][e]));
      }
  }
};
// The pulled leaves' cells (positions below lo1); P rows of the others.  The
// gates are the product's rows: lane (r, g) holds units 16 wm + 4 g .. + 3 of
// pulled rows 64 wn + 4 r + c, every gate, and writes 16 bytes at a time (with
// the pulled rows as the product's rows, 4-byte stores: 286 us instead of 276
// on 21 000 leaves, D = 300, at H = 1024, 122 instead of 101 on 18 900 at 512).
struct X3PullOut {
  int rows, lo1, with_f;
  __device__ void operator()(const Net& n, int, int g0, int m0, int wm, int wn, int g, int r,
                             const v4f (&acc)[4][4]) const {
    const int H = n.H, u = g0 / 4 + 16 * wm + 4 * g;
    Bias4 b;
    lstm_bias4(n, u, b);
    const float bi[4] = {b.i.x, b.i.y, b.i.z, b.i.w}, bo[4] = {b.o.x, b.o.y, b.o.z, b.o.w};
    const float bu[4] = {b.u.x, b.u.y, b.u.z, b.u.w};
    auto f4 = [](const float (&x)[4]) { return make_float4(x[0], x[1], x[2], x[3]); };
    auto v4 = [](const v4f& x) { return make_float4(x[0], x[1], x[2], x[3]); };
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int m = m0 + 64 * wn + 4 * r + c;
      if (m >= rows) continue;
      const int p = n.pull_list[m];
      const v4f zi = acc[G_I][c], zo = acc[G_O][c], zu = acc[G_U][c];
      if (p < lo1) {
        float ig[4], og[4], ug[4], cc[4], h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ig[e] = sigmoidf_(zi[e] + bi[e]);
          og[e] = sigmoidf_(zo[e] + bo[e]);
          ug[e] = tanh_(zu[e] + bu[e]);
          cc[e] = ig[e] * ug[e];
          h[e] = og[e] * tanh_(cc[e]);
        }
        st4(n.Hs + (size_t)p * H + u, f4(h));
        st4(n.Cs + (size_t)p * H + u, f4(cc));
        if (n.Gs) {   // a leaf's forget gates are never read; null in inference
          float* gs = n.Gs + (size_t)p * n.GW + u;
          st4(gs, f4(ig));
          st4(gs + 2 * H, f4(og));
          st4(gs + 3 * H, f4(ug));
        }
        const int v = n.order[p];
        st4(n.h_out + (size_t)v * H + u, f4(h));
        if (n.c_out) st4(n.c_out + (size_t)v * H + u, f4(cc));
      } else {
        float* P = n.P + (size_t)p * 4 * H + u;
        st4(P + G_I * H, v4(zi));
        if (with_f) st4(P + G_F * H, v4(acc[G_F][c]));
        st4(P + G_O * H, v4(zo));
        st4(P + G_U * H, v4(zu));
      }
    }
  }
};

// The sum over k in [z kchunk, (z + 1) kchunk) of A B^T into ep; the tile and
// its pipeline as in k_x3_tn (lazy.hip).  PARTS: 3 (split fp32) or 1 (bf16).
// Items: bands of kX3Band column tiles, a band's row tiles one after the other,
// a contiguous eighth to each XCD: the 96 tiles that an XCD has in flight are
// then about 8 x 12 and share their operands' rows in its L2.  WGS workgroups
// share a CU.
constexpr int kX3Band = 8;
template <class LA, class LB, class EP, int PARTS, int BLOCKS, int WGS>
__global__ void __launch_bounds__(256, WGS) k_x3_gemm(Net n, LA la, LB lb, EP ep, int ty, int tx,
                                                      int K, int kchunk, int items) {
  constexpr int OPB = PARTS * kX3Plane;
  __shared__ __attribute__((aligned(16))) char lds[2 * OPB];
  const int item = xcd_item(blockIdx.x, items);
  if (item < 0) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wm = w & 1, wn = w >> 1, z = item / (tx * ty), it = item % (tx * ty);
  const int band = it / (kX3Band * ty), in = it % (kX3Band * ty);
  const int bw = min(kX3Band, tx - band * kX3Band);
  const int m0 = in / bw * kX3Tile, n0 = (band * kX3Band + in % bw) * kX3Tile;
  const int klo = z * kchunk, khi = min(K, klo + kchunk);
  const bool bside = __builtin_amdgcn_readfirstlane(tid >> 7) != 0;
  v4f acc[4][4];
  auto sum = [&](auto parts, int t, auto&& mma) {
    constexpr int P = decltype(parts)::value;
    typename LA::State sa{};
    typename LB::State sb{};
    if (bside) lb.init(n, sb, t, n0);
    else la.init(n, sa, t, m0);
    float4 v[8];
    auto load = [&](int k0) {
      if (bside) lb.load(n, sb, k0, khi, v);
      else la.load(n, sa, k0, khi, v);
    };
    zero_acc(acc);
    if (klo < khi) load(klo);
    for (int k0 = klo; k0 < khi; k0 += kBK) {
      if (k0 > klo) __syncthreads();   // the previous chunk's fragments are read
      if (bside) LB::template store<P>(lds + OPB, sb, v);
      else LA::template store<P>(lds, sa, v);
      __syncthreads();
      if (k0 + kBK < khi) load(k0 + kBK);
      __builtin_amdgcn_sched_barrier(0);   // the next chunk's loads go out before these products
      mma();
    }
  };
  sum(std::integral_constant<int, PARTS>{}, tid & 127,
      [&] { x3_mma<PARTS, BLOCKS>(lds, lds + OPB, wm, wn, acc); });
  if constexpr (PARTS == 3)
    if (x3_nan(acc))   // NaN, or an operand without parts (split3.h)
      sum(std::integral_constant<int, 0>{}, x3_again(tid & 127),
          [&] { x3_mma_f32(lds, lds + OPB, wm, wn, acc); });
  ep(n, z, m0, n0, wm, wn, g, r, acc);
}

template <int PARTS, int BLOCKS, int WGS, class LA, class LB, class EP>
void x3_gemm(const char* name, const Net& n, LA la, LB lb, EP ep, int M, int Nc, int K, int kchunk,
             hipStream_t s) {
  const int ty = cdiv(M, kX3Tile), tx = cdiv(Nc, kX3Tile);
  const int items = tx * ty * (K > 0 ? cdiv(K, kchunk) : 1);
  CAVS_LAUNCH(name, (k_x3_gemm<LA, LB, EP, PARTS, BLOCKS, WGS>), dim3(xcd_grid(items)), dim3(256), 0,
              s, n, la, lb, ep, ty, tx, K, kchunk, items);
}

// A bf16 forward level: 32 units x 128 positions a workgroup, wavefronts 2 x 2
// of 16 x 64.  LDS block j of A is gate block j of the units (the rounded U^T),
// B one plane per operand: h~ (rounded after the sum) and each child's h; i, o
// and u multiply the first, f_k plane k + 1.  Two chunks' loads are in flight
// and two LDS buffers take one barrier a chunk: a CU's only workgroup spends
// 1.3 us a chunk (one chunk ahead: 1.5), a full chip 255 TFLOP/s (3652 rows, H =
// 1024: 145 us, 177 in 64 x 32 tiles that stage fp32 operands); bound by
// latency and the operands' way through L2, each element being used for 32
// units or 128 rows.
template <int NCH>
__global__ void __launch_bounds__(256, 2) k_lstm_fwd_bf(Net n, int off, int M, int ty, int tx,
                                                        int items) {
  constexpr int NB = NCH == 1 ? 1 : 1 + NCH;
  __shared__ __attribute__((aligned(16))) char lds[2][(1 + NB) * kX3Plane];
  const int item = xcd_item(blockIdx.x, items);
  if (item < 0) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wm = w & 1, wn = w >> 1, H = n.H;
  const int band = item / (kX3Band * ty), in = item % (kX3Band * ty);
  const int bw = min(kX3Band, tx - band * kX3Band);
  const int u0 = in / bw * 32, r0 = (band * kX3Band + in % bw) * kX3Tile;
  // LDS rows R and R + 64, octet oq of both operands
  const int oq = tid & 3, R = tid >> 2;
  const float* src[2][NCH];
  const u16* wsrc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = R + 64 * i, p = off + min(r0 + 4 * (row & 31) + (row >> 5), M - 1);
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int c = n.child_pos[(size_t)p * NCH + k];
      src[i][k] = (c >= 0 ? n.Hs + (size_t)c * H : n.zrow) + 8 * oq;
    }
    wsrc[i] = n.UTb + ((size_t)(row >> 5) * H + u0 + (row & 31)) * H + 8 * oq;
  }
  struct Stage {
    float4 v[2][NCH][2];
    bf16x8 w[2];
  } st[2];
  auto load = [&](Stage& x, int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int k = 0; k < NCH; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) x.v[i][k][h] = ldg4(src[i][k] + k0 + 4 * h);
      x.w[i] = *reinterpret_cast<const bf16x8*>(wsrc[i] + k0);
    }
  };
  auto pack = [](const float4& a, const float4& b) {
    return make_uint4(f2bf2(a.x, a.y), f2bf2(a.z, a.w), f2bf2(b.x, b.y), f2bf2(b.z, b.w));
  };
  auto store = [&](const Stage& x, char* buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      char* d = buf + x3_addr(R + 64 * i, oq);
      *reinterpret_cast<bf16x8*>(d) = x.w[i];
      float4 s0 = x.v[i][0][0], s1 = x.v[i][0][1];
#pragma unroll
      for (int k = 1; k < NCH; ++k) {
        s0 = add4(s0, x.v[i][k][0]);
        s1 = add4(s1, x.v[i][k][1]);
      }
      *reinterpret_cast<uint4*>(d + kX3Plane) = pack(s0, s1);
      if constexpr (NCH > 1) {
#pragma unroll
        for (int k = 0; k < NCH; ++k)
          *reinterpret_cast<uint4*>(d + (2 + k) * kX3Plane) = pack(x.v[i][k][0], x.v[i][k][1]);
      }
    }
  };
  v4f acc[3 + NCH][4];
#pragma unroll
  for (int a = 0; a < 3 + NCH; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = v4f{0.f, 0.f, 0.f, 0.f};
  load(st[0], 0);
  __builtin_amdgcn_sched_barrier(0);   // in this order, or the loop waits for both
  load(st[1], kBK);
  __builtin_amdgcn_sched_barrier(0);
  for (int k0 = 0; k0 < H; k0 += 2 * kBK) {   // H is a multiple of 64
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      // a buffer's readers are past the barrier of the other's chunk; left to
      // itself the compiler waits for both stages' loads here
      __builtin_amdgcn_sched_barrier(0);
      store(st[s], lds[s]);
      __syncthreads();
      load(st[s], min(k0 + (s + 2) * kBK, H - kBK));   // past the end: the last chunk, unused
      __builtin_amdgcn_sched_barrier(0);   // the loads go out before these products
      auto frag = [&](int plane, int row) {
        return *reinterpret_cast<const bf16x8*>(lds[s] + plane * kX3Plane + x3_addr(row, g));
      };
      bf16x8 a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = frag(0, 32 * j + 16 * wm + r);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int row = 32 * c + 16 * wn + r;
        const bf16x8 b = frag(1, row);
        acc[G_I][c] = mfma_bf16_16x16x32(a[G_I], b, acc[G_I][c]);
        acc[G_O][c] = mfma_bf16_16x16x32(a[G_O], b, acc[G_O][c]);
        acc[G_U][c] = mfma_bf16_16x16x32(a[G_U], b, acc[G_U][c]);
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
          v4f& f = acc[k == 0 ? G_F : 3 + k][c];
          f = mfma_bf16_16x16x32(a[G_F], NCH == 1 ? b : frag(2 + k, row), f);
        }
      }
    }
  }
  const int u = u0 + 16 * wm + 4 * g;
  Bias4 b;
  lstm_bias4(n, u, b);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int m = r0 + 64 * wn + 4 * r + c;
    if (m >= M) continue;
    FwdPos<NCH> q;
    FwdCell4<NCH> e;
    lstm_fwd_pos<NCH>(n, off + m, q);
    lstm_fwd_cell4<NCH>(n, q, u, e);
    v4f zf[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) zf[k] = acc[k == 0 ? G_F : 3 + k][c];
    lstm_fwd_fin4<NCH>(n, off + m, u, q, b, e, acc[G_I][c], acc[G_O][c], acc[G_U][c], zf);
  }
}

}  // namespace

void lstm_fwd_bf(const Net& n, int off, int M, hipStream_t s) {
  const int ty = n.H / 32, tx = cdiv(M, kX3Tile), items = tx * ty;
  if (n.N == 1)
    CAVS_LAUNCH_ROWS("k_lstm_fwd_bf<1>", off, M, k_lstm_fwd_bf<1>, dim3(xcd_grid(items)), dim3(256), 0, s, n, off,
                M, ty, tx, items);
  else
    CAVS_LAUNCH_ROWS("k_lstm_fwd_bf<2>", off, M, k_lstm_fwd_bf<2>, dim3(xcd_grid(items)), dim3(256), 0, s, n, off,
                M, ty, tx, items);
}

// Z[V, C] = h W_s: W_s as it is ([H, C], k-major).  2275 x 10 000 x 512:
// 233 us on fp32 instructions (and 16 us of transposing W_s) -> 135 us.
void lm_logits(const Net& n, hipStream_t s) {
  x3_gemm<3, 15, 3>("k_x3_gemm<lm_logits>", n, X3Rows{n.Hs, n.H, n.V}, X3Cols{n.Ws, n.C, n.C},
                    X3Out{n.dZ, n.C, n.V, n.C}, n.V, n.C, n.H, n.H, s);
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
  x3_gemm<3, 15, 2>("k_x3_gemm<lm_dh>", n, X3Rows{n.dZ, n.C, n.V}, X3Rows{n.Ws, n.C, n.H},
                    X3Out{S > 1 ? part : n.dHL, n.H, n.V, n.H}, n.V, n.H, n.C, kchunk, s);
  if (S == 1) return;
  SplitJobs jobs;
  jobs.j[jobs.n++] = SplitJob{part, n.dHL, S, n.V, n.H, n.H, 0, 1 << 30, 0};
  reduce_split_jobs(jobs, s);
}

template <int PARTS>
static void x3_pull(const char* n4, const char* n3, const Net& n, int n_pull, bool with_f, int lo1,
                    hipStream_t s) {
  constexpr int WGS = PARTS == 1 ? 3 : 2;
  std::conditional_t<PARTS == 1, X3GatesK, X3Gates> gates{};
  if (with_f)
    x3_gemm<PARTS, 15, WGS>(n4, n, gates, X3Pulled{{nullptr, 0, n_pull}},
                            X3PullOut{n_pull, lo1, 1}, 4 * n.H, n_pull, n.D, n.D, s);
  else   // i|o|u: the f block is neither formed nor stored
    x3_gemm<PARTS, 13, WGS>(n3, n, gates, X3Pulled{{nullptr, 0, n_pull}},
                            X3PullOut{n_pull, lo1, 0}, 4 * n.H, n_pull, n.D, n.D, s);
}

// fp32: from a tile per CU up (4 867 leaves, D = 300, H = 512, 624 tiles: 65 ->
// 50 us; 3 581 rows, D = H = 512, 448 tiles: 80 -> 54; 288 tiles: 61 -> 49).
// Below that the 64 x 32 tiles of k_pull_tile fill the chip better (144 tiles:
// 30 against 29 us, 120 tiles, D = 100: 13 against 18).
bool x3_pull_applies(const Net& n, int n_pull) {
  return n.bf || cdiv(4 * n.H, kX3Tile) * cdiv(n_pull, kX3Tile) >= 256;
}

// The pull product with the pulled leaves' cells in its epilogue (six rows of H
// written each: bound by memory).  bf16, 21 004 leaves, D = 300, H = 1024: pull
// and leaf kernels 246 + 164 us -> 248 (520 MB of stores alone are 100 us at the
// rate of a large copy); 18 901 at 512, inference: 167 -> 88.
void pull_gemm_x3(const Net& n, int n_pull, bool with_f, int lo1, hipStream_t s) {
  if (n.bf)
    x3_pull<1>("k_x3_gemm<pull4, bf16>", "k_x3_gemm<pull3, bf16>", n, n_pull, with_f, lo1, s);
  else
    x3_pull<3>("k_x3_gemm<pull4>", "k_x3_gemm<pull3>", n, n_pull, with_f, lo1, s);
}

// bf16 dX of many rows (dx_gemm, lazy.hip, draws the line to k_dx_gemm_bf's 64 x
// 64 tiles): 21 004 x 300 x 3072, 216 us in 32 x 64 tiles, 130 here.  Not in fp32:
// the contraction is 3H or more deep and the tiles few, so a tile's chain of
// chunks is what counts (4 867 x 300 x 1536: 46 us in 32 x 64 tiles, 102 here).
void dx_gemm_bf(const Net& n, int n_pull, bool with_f, float* dX, hipStream_t s) {
  const X3Rows rows{nullptr, 0, n_pull}, wx{n.Wx, 4LL * n.H, n.D};
  const int K = (with_f ? 4 : 3) * n.H;
  x3_gemm<1, 15, 3>("k_x3_gemm<dX, bf16>", n, X3DxA{rows, (int)with_f}, X3DxB{wx, (int)with_f},
                    X3DxOut{dX, n_pull}, n_pull, n.D, K, K, s);
}

}  // namespace cavs

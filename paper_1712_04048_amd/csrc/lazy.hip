// Operators that are not on a gather->scatter path of F or dF and therefore
// run batched over all vertices at once (lazy batching, Section 3.5), plus
// the eager pull projection:
//   - pull:   P = X W_x for every vertex that pulls an input (one GEMM);
//   - push:   the loss head over every labelled vertex (z = h W_s + b_s);
//   - dF:     dW_x, dU, db, dX, dW_s, db_s as long-K products over all
//             vertices, with deterministic split-K (fixed-order reduction).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "lds_ring.h"
#include "lstm_dev.h"
#include "split3.h"

namespace cavs {
namespace {

constexpr int kMaxSplits = 16;   // sizes the split-K scratch: 16 x (4H x H) floats
constexpr int kSplitCap = 32;    // more splits only where the scratch holds them

// ------------------------------------------------------------- pull GEMM
// Pull projection P = x W_x fused with the cell of the pulled leaves: each
// lane holds all NG gate blocks (i|o|u when no vertex with children pulls,
// else i|f|o|u) of its row and units.  A leaf row (position below lo1)
// finishes its cell here (h, c, saved gates, outputs); any other pulled row
// stores its P row for the level epilogue.  On the direct-to-LDS ring of the
// level tiles: a
// workgroup owns 64 pulled rows x 32 units x NG gate blocks.  Stage rows:
// the 64 x rows (gathered through pull_list and pull_pos), then the rows of
// W_x^T for each gate block's 32 units; chunks past D read the zero row.
// Four wavefronts as 2 x 2 (32 rows x 16 units each); the weight fragment
// is the MFMA's A operand, so a lane holds four consecutive units of one
// row (float4 epilogue).  Fragments are double-buffered in registers.
template <int NG, int BM, int S>
__global__ void __launch_bounds__(256) k_pull_tile(Net n, int n_pull, int lo1) {
  constexpr int BU = 32, TM = BM / 32;
  constexpr int ROWS = BM + NG * BU, IPW = ROWS / 32;
  static_assert(IPW * 32 == ROWS && S >= 2 && S <= 4, "tile shape");
  __shared__ __attribute__((aligned(1024))) float L0[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L1[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L2[S > 2 ? ROWS * 32 : 4];
  __shared__ __attribute__((aligned(1024))) float L3[S > 3 ? ROWS * 32 : 4];
  const Ring<ROWS, S> ring{L0, L1, L2, L3};
  const int H = n.H, H4 = 4 * H, D = n.D;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int wr = w & 1, wu = w >> 1;
  int rt, ut;
  xcd_tile(H / BU, rt, ut);
  const int m0 = rt * BM, u0 = ut * BU;
  auto gcol = [](int g) { return NG == 4 ? g : (g == 0 ? G_I : g + 1); };

  // epilogue operands first: the position and vertex of each row, the bias
  const int j0 = u0 + wu * 16 + 4 * gq;
  int pos[TM], vid[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int m = m0 + wr * (BM / 2) + tm * 16 + r;
    pos[tm] = m < n_pull ? n.pull_list[m] : -1;
    vid[tm] = pos[tm] >= 0 && pos[tm] < lo1 ? n.order[pos[tm]] : 0;
  }
  Bias4 bias;
  lstm_bias4(n, j0, bias);

  const float* src[IPW];
  int kq[IPW];
#pragma unroll
  for (int t = 0; t < IPW; ++t) {
    const int row = (w * IPW + t) * 8 + (lane >> 3), qg = (lane & 7) ^ (row & 7);
    kq[t] = 4 * qg;
    if (row < BM) {
      const int p = n.pull_list[min(m0 + row, n_pull - 1)];
      src[t] = n.X + (size_t)n.pull_pos[p] * D + 4 * qg;
    } else {
      const int b = row - BM, g = b / BU, u = b % BU;
      src[t] = n.WxT + (size_t)(gcol(g) * H + u0 + u) * D + 4 * qg;
    }
  }
  const int wofs = __builtin_amdgcn_readfirstlane(w * IPW * 256);
  v4f acc[TM][NG];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[tm][g] = v4f{0.f, 0.f, 0.f, 0.f};

  auto issue = [&](auto sc, int c) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr_of(ring.at(sc)) + 4u * wofs);
    const int k0 = c * kBK;
#pragma unroll
    for (int t = 0; t < IPW; ++t)
      copy16_to_lds(k0 + kq[t] < D ? src[t] + k0 : n.zrow, base + 1024u * t);
  };
  struct Frag {
    float a[TM][8], b[NG][8];
  };
  auto read = [&](const float* Ls, Frag& f) {
#pragma unroll
    for (int g = 0; g < NG; ++g) frag_sw(Ls, BM + g * BU + wu * 16 + r, gq, f.b[g]);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) frag_sw(Ls, wr * (BM / 2) + tm * 16 + r, gq, f.a[tm]);
  };
  auto body = [&](const float* Lnext, Frag& cur, Frag& nxt, int) {
    read(Lnext, nxt);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int g = 0; g < NG; ++g) acc[tm][g] = mfma_chunk8<false>(cur.b[g], cur.a[tm], acc[tm][g]);
    interleave_reads<2 * (NG + TM), TM * NG * 8>();
  };
  ring_loop_db<S, IPW, Frag>((D + kBK - 1) / kBK, ring, issue, read, body);

#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int p = pos[tm];
    if (p < 0) continue;
    if (p < lo1) {
      const v4f zi = acc[tm][0], zo = acc[tm][NG == 4 ? 2 : 1], zu = acc[tm][NG == 4 ? 3 : 2];
      const float bi[4] = {bias.i.x, bias.i.y, bias.i.z, bias.i.w};
      const float bo[4] = {bias.o.x, bias.o.y, bias.o.z, bias.o.w};
      const float bu[4] = {bias.u.x, bias.u.y, bias.u.z, bias.u.w};
      float ig[4], og[4], ug[4], c[4], h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ig[e] = sigmoidf_(zi[e] + bi[e]);
        og[e] = sigmoidf_(zo[e] + bo[e]);
        ug[e] = tanh_(zu[e] + bu[e]);
        c[e] = ig[e] * ug[e];
        h[e] = og[e] * tanh_(c[e]);
      }
      auto f4 = [](const float (&x)[4]) { return make_float4(x[0], x[1], x[2], x[3]); };
      st4(n.Hs + (size_t)p * H + j0, f4(h));
      st4(n.Cs + (size_t)p * H + j0, f4(c));
      if (n.Gs) {   // a leaf's forget gates are never read; null in inference
        float* gs = n.Gs + (size_t)p * n.GW + j0;
        st4(gs, f4(ig));
        st4(gs + 2 * H, f4(og));
        st4(gs + 3 * H, f4(ug));
      }
      st4(n.h_out + (size_t)vid[tm] * H + j0, f4(h));
      if (n.c_out) st4(n.c_out + (size_t)vid[tm] * H + j0, f4(c));
    } else {
#pragma unroll
      for (int g = 0; g < NG; ++g)
        st4(n.P + (size_t)p * H4 + gcol(g) * H + j0,
            make_float4(acc[tm][g][0], acc[tm][g][1], acc[tm][g][2], acc[tm][g][3]));
    }
  }
}

// ------------------------------------- long-K "A^T B" products, bf16 operands
// out[s][m][n] = sum_{q in split s} A(q, m) B(q, n).  The loader supplies
// 4 consecutive m (or n) of row q; rows outside [0, Q) are never requested.
// bf16 vertices have one or two child slots.
struct LdDUiou {  // dU[:, i|o|u] (or all four blocks when N == 1): A = h~, B = dA
  static constexpr const char* kNameBf = "k_tn_gemm_bf<LdDUiou>";
  static constexpr const char* kNamePack = "k_pack_bf<LdDUiou>";
  static constexpr const char* kNameNt = "k_nt_bf<LdDUiou>";
  struct Idx {
    int c0, c1;
  };
  Net n;
  int off1;
  __device__ Idx idx(int q) const {
    const int p = off1 + q;
    return {n.child_pos[(size_t)p * n.N], n.N == 2 ? n.child_pos[(size_t)p * n.N + 1] : -1};
  }
  __device__ float4 a4(const Idx& x, int q, int m) const {
    float4 s = x.c0 >= 0 ? ldg4(n.Hs + (size_t)x.c0 * n.H + m) : f4zero();
    if (x.c1 >= 0) s = add4(s, ldg4(n.Hs + (size_t)x.c1 * n.H + m));
    return s;
  }
  __device__ float4 b4(const Idx&, int q, int c) const {
    const int p = off1 + q;
    const int col = (n.N == 2 && c >= n.H) ? c + n.H : c;
    return ldg4(n.dA + (size_t)p * n.GW + col);
  }
};

struct LdDUf {  // dU[:, f], two child slots: q in [0, 2 MI), A = h_k, B = dA_fk
  static constexpr const char* kNameBf = "k_tn_gemm_bf<LdDUf>";
  static constexpr const char* kNamePack = "k_pack_bf<LdDUf>";
  static constexpr const char* kNameNt = "k_nt_bf<LdDUf>";
  struct Idx {
    int cp;
  };
  Net n;
  int off1, MI;
  __device__ Idx idx(int q) const {
    const int k = q / MI, p = off1 + q - k * MI;
    return {n.child_pos[(size_t)p * n.N + k]};
  }
  __device__ float4 a4(const Idx& x, int q, int m) const {
    return x.cp >= 0 ? ldg4(n.Hs + (size_t)x.cp * n.H + m) : f4zero();
  }
  __device__ float4 b4(const Idx&, int q, int c) const {
    const int k = q / MI, p = off1 + q - k * MI;
    return ldg4(n.dA + (size_t)p * n.GW + f_col(k, n.H) + c);
  }
};

struct LdDWx {  // dW_x: q over pulling vertices, A = x, B = dA_x (f = the sum of the f_k)
  static constexpr const char* kNameBf = "k_tn_gemm_bf<LdDWx>";
  static constexpr const char* kNamePack = "k_pack_bf<LdDWx>";
  static constexpr const char* kNameNt = "k_nt_bf<LdDWx>";
  struct Idx {
    int p, row;
  };
  Net n;
  int with_f;
  __device__ Idx idx(int q) const {
    const int p = n.pull_list[q];
    return {p, n.pull_pos[p]};
  }
  __device__ float4 a4(const Idx& x, int q, int m) const {
    return m < n.D ? ldg4(n.X + (size_t)x.row * n.D + m) : f4zero();
  }
  __device__ float4 b4(const Idx& x, int q, int c) const {
    const int H = n.H;
    const int col = (with_f || c < H) ? c : c + H;
    const float* row = n.dA + (size_t)x.p * n.GW;
    float4 v = ldg4(row + col);
    if (col >= H && col < 2 * H)
      for (int k = 1; k < n.N; ++k) v = add4(v, ldg4(row + (2 + k) * H + col));
    return v;
  }
};

// dX[pull_pos[p], d] = sum over the gate columns of dA[p] W_x[d] through the
// LDS ring (lds_ring.h): i|o|u, or with_f all 3 + N blocks of the dA row, the
// forget block of every child slot against the one f block of W_x (the sum
// over slots joins the contraction, which a row of pre-summed columns would
// take another pass to form).  A workgroup owns BM pulled rows x BN input
// columns; stage rows [0, BM) are dA rows (gathered through pull_list),
// [BM, BM + BN) rows of W_x.  Rows
// past n_pull or D read the last valid row; their products are not stored.
// SLOTS: with_f and several child slots.  The chain is then (3 + N) H deep
// instead of 4H, so even and odd chunks are summed apart: relative error of dX
// against 64 bits 4.2e-7 with the slots summed before the product, 5.1e-7 in
// one chain, 3.8e-7 so (H = 320, two slots).
template <int BM, int BN, int S, bool SLOTS>
__global__ void __launch_bounds__(256) k_dx_tile(Net n, int n_pull, int with_f, float* dX) {
  constexpr int TM = BM / 32, TN = BN / 32, ROWS = BM + BN, IPW = ROWS / 32;
  static_assert(IPW * 32 == ROWS && S >= 2 && S <= 4, "tile shape");
  __shared__ __attribute__((aligned(1024))) float L0[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L1[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L2[S > 2 ? ROWS * 32 : 4];
  __shared__ __attribute__((aligned(1024))) float L3[S > 3 ? ROWS * 32 : 4];
  const Ring<ROWS, S> ring{L0, L1, L2, L3};
  const int H = n.H, H4 = 4 * H, D = n.D, GW = n.GW;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int wr = w & 1, wn = w >> 1;
  const int m0 = blockIdx.x * BM, d0 = blockIdx.y * BN;
  // output rows of this lane (one per row block), fetched before the product
  int orow[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int m = m0 + wr * (BM / 2) + tm * 16 + r;
    orow[tm] = m < n_pull ? n.pull_pos[n.pull_list[m]] : -1;
  }
  const float* src[IPW];
  bool isw[IPW];
#pragma unroll
  for (int t = 0; t < IPW; ++t) {
    const int row = (w * IPW + t) * 8 + (lane >> 3), qg = (lane & 7) ^ (row & 7);
    const float* ptr;
    isw[t] = row >= BM;
    if (row < BM) ptr = n.dA + (size_t)n.pull_list[min(m0 + row, n_pull - 1)] * GW;
    else ptr = n.Wx + (size_t)min(d0 + row - BM, D - 1) * H4;
    src[t] = ptr + 4 * qg;
  }
  const int wofs = __builtin_amdgcn_readfirstlane(w * IPW * 256);
  v4f acc[TM][TN], odd[TM][TN];
  zero_acc(acc);
  if constexpr (SLOTS) zero_acc(odd);
  auto issue = [&](auto sc, int c) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr_of(ring.at(sc)) + 4u * wofs);
    const int k0 = c * kBK, acol = (with_f || k0 < H) ? k0 : k0 + H;
    if constexpr (SLOTS) {
      // f_1, f_2, f_3 (columns 4H, 5H, 6H ..): W_x's f block again
      const int wcol = k0 < H4 ? k0 : k0 - 3 * H - (k0 >= 5 * H ? H : 0) - (k0 >= 6 * H ? H : 0);
#pragma unroll
      for (int t = 0; t < IPW; ++t) copy16_to_lds(src[t] + (isw[t] ? wcol : k0), base + 1024u * t);
    } else {
#pragma unroll
      for (int t = 0; t < IPW; ++t) copy16_to_lds(src[t] + acol, base + 1024u * t);
    }
  };
  struct Frag {
    float a[TM][8], b[TN][8];
  };
  auto read = [&](const float* Ls, Frag& f) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) frag_sw(Ls, BM + wn * (BN / 2) + tn * 16 + r, gq, f.b[tn]);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) frag_sw(Ls, wr * (BM / 2) + tm * 16 + r, gq, f.a[tm]);
  };
  // A = W_x fragment (d), B = dA fragment (rows): a lane holds four
  // consecutive d of one row
  auto body = [&](const float* Lnext, Frag& cur, Frag& nxt, int c) {
    read(Lnext, nxt);
    auto& to = SLOTS && (c & 1) ? odd : acc;   // known at compile time in the unrolled steps
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) to[tm][tn] = mfma_chunk8<false>(cur.b[tn], cur.a[tm], to[tm][tn]);
    interleave_reads<2 * (TM + TN), TM * TN * 8>();
  };
  ring_loop_db<S, IPW, Frag>((with_f ? GW : 3 * H) / kBK, ring, issue, read, body);
  if constexpr (SLOTS) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) acc[tm][tn] += odd[tm][tn];
  }
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    if (orow[tm] < 0) continue;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int d = d0 + wn * (BN / 2) + tn * 16 + 4 * gq;
      if (d < D)   // D % 4 == 0: the four d are all in range or all out
        st4(dX + (size_t)orow[tm] * D + d,
            make_float4(acc[tm][tn][0], acc[tm][tn][1], acc[tm][tn][2], acc[tm][tn][3]));
    }
  }
}

// ------------------------------------------------------------ bf16 variants
// Operands are rounded to bf16 while they are staged into LDS (k-contiguous
// rows), accumulation is fp32.
// dX of few pulled rows: 64 x 64 tiles.  While the chip is not full a launch
// takes as long as one tile's chain of chunks, and a chunk is shorter here than
// in the 128 x 128 tiles of dx_gemm_bf (x3.hip): H = 1024, D = 300, 64 rows 75
// against 97 us, 4 800 109 / 124, 12 000 (940 workgroups) 123 / 142, 16 000
// (1 250) 190 / 148.
__global__ void __launch_bounds__(256) k_dx_gemm_bf(Net n, int n_pull, int with_f, float* dX) {
  constexpr int BM = 64, BN = 64;
  __shared__ __attribute__((aligned(16))) u16 As[BM * kLDH];
  __shared__ __attribute__((aligned(16))) u16 Bs[BN * kLDH];
  const int H = n.H, H4 = 4 * H, D = n.D, GW = n.GW, N = n.N;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int wrow = (w >> 1) * 32, wcol = (w & 1) * 32;
  const int m0 = blockIdx.x * BM, d0 = blockIdx.y * BN;
  const float* asrc[2];
  int arow[2], aq[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int idx = tid + 256 * a;
    arow[a] = idx / 8;
    aq[a] = idx % 8;
    asrc[a] = m0 + arow[a] < n_pull ? n.dA + (size_t)n.pull_list[m0 + arow[a]] * GW : nullptr;
  }
  float4 ra[2], rb[2];
  auto col_of = [&](int kc) {
    const int c = kc * kBK;
    if (with_f) return c;
    return c < H ? c : c + H;
  };
  auto gload = [&](int kc) {
    const int c0 = col_of(kc);
    const bool fblock = c0 >= H && c0 < 2 * H;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      float4 v = f4zero();
      if (asrc[a]) {
        v = ldg4(asrc[a] + c0 + 4 * aq[a]);
        if (fblock && N == 2) v = add4(v, ldg4(asrc[a] + 3 * H + c0 + 4 * aq[a]));
      }
      ra[a] = v;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int idx = tid + 256 * b, dr = idx / 8, q = idx % 8;
      rb[b] = d0 + dr < D ? ldg4(n.Wx + (size_t)(d0 + dr) * H4 + c0 + 4 * q) : f4zero();
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int a = 0; a < 2; ++a) st_bf4(&As[arow[a] * kLDH + 4 * aq[a]], ra[a]);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int idx = tid + 256 * b;
      st_bf4(&Bs[(idx / 8) * kLDH + 4 * (idx % 8)], rb[b]);
    }
  };
  v4f acc[2][2];
  zero_acc(acc);
  const int nk = (with_f ? H4 : 3 * H) / kBK;
  gload(0);
  for (int kc = 0; kc < nk; ++kc) {
    __syncthreads();
    sstore();
    __syncthreads();
    if (kc + 1 < nk) gload(kc + 1);
    mfma_chunk_bf<2, 2>(As, Bs, wrow, wcol, acc);
  }
#pragma unroll
  for (int tm = 0; tm < 2; ++tm)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + wrow + tm * 16 + 4 * gq + i;
      if (m >= n_pull) continue;
      const int row = n.pull_pos[n.pull_list[m]];
#pragma unroll
      for (int tn = 0; tn < 2; ++tn) {
        const int d = d0 + wcol + tn * 16 + r;
        if (d < D) dX[(size_t)row * D + d] = acc[tm][tn][i];
      }
    }
}

template <class L>
__global__ void __launch_bounds__(256) k_tn_gemm_bf(L ld, int Q, int qchunk, int Mo, int No,
                                                    float* out) {
  constexpr int BM = 64, BN = 64;
  __shared__ __attribute__((aligned(16))) u16 As[BM * kLDH];
  __shared__ __attribute__((aligned(16))) u16 Bs[BN * kLDH];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int wrow = (w >> 1) * 32, wcol = (w & 1) * 32;
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM, s = blockIdx.z;
  const int q_lo = s * qchunk, q_hi = min(Q, q_lo + qchunk);
  float4 ra[2], rb[2];
  auto gload = [&](int q0) {
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int idx = tid + 256 * a, qq = idx / 16, c4 = idx % 16;
      const int q = q0 + qq;
      if (q < q_hi) {
        const typename L::Idx ix = ld.idx(q);
        ra[a] = m0 + 4 * c4 < Mo ? ld.a4(ix, q, m0 + 4 * c4) : f4zero();
        rb[a] = ld.b4(ix, q, n0 + 4 * c4);
      } else {
        ra[a] = f4zero();
        rb[a] = f4zero();
      }
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int idx = tid + 256 * a, qq = idx / 16, c4 = idx % 16;
      st_bf4_t(&As[(4 * c4) * kLDH + qq], kLDH, ra[a]);
      st_bf4_t(&Bs[(4 * c4) * kLDH + qq], kLDH, rb[a]);
    }
  };
  v4f acc[2][2];
  zero_acc(acc);
  gload(q_lo);
  for (int q0 = q_lo; q0 < q_hi; q0 += kBK) {
    __syncthreads();
    sstore();
    __syncthreads();
    if (q0 + kBK < q_hi) gload(q0 + kBK);
    mfma_chunk_bf<2, 2>(As, Bs, wrow, wcol, acc);
  }
  float* o = out + (size_t)s * Mo * No;
#pragma unroll
  for (int tm = 0; tm < 2; ++tm)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + wrow + tm * 16 + 4 * gq + i;
      if (m >= Mo) continue;
#pragma unroll
      for (int tn = 0; tn < 2; ++tn) o[(size_t)m * No + n0 + wcol + tn * 16 + r] = acc[tm][tn][i];
    }
}

// dst[m, col(n)] = sum_s part[s][m][n] in split order; col(n) = col_off + n
// (+ gap for n >= gap_start).
__global__ void k_reduce_splits(const float* __restrict__ part, int S, int Mo, int No,
                                float* __restrict__ dst, int ldd, int col_off, int gap_start,
                                int gap) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)Mo * No) return;
  const int m = (int)(idx / No), nn = (int)(idx % No);
  float s = 0.f;
  for (int k = 0; k < S; ++k) s += part[(size_t)k * Mo * No + idx];
  dst[(size_t)m * ldd + col_off + nn + (nn >= gap_start ? gap : 0)] = s;
}

// ------------------------------------------ long-K "A^T B" products, split
// out[s][m][n] = sum over q in split s of A[q][m] B[q][n]: the lazily batched
// weight gradients.  Row q of A and of B are rows of the level-major buffers
// (h, h~, x, dA, delta, dZ) at element offsets that depend on the product.
enum TnKind : int {
  TN_DU = 0,    // dU: A = h~ (one child slot: the child's h), B = dA, q an internal position
  TN_DUF = 1,   // dU[:, f]: A = h_k, B = dA_fk, q = k MI + internal position
  TN_DWX = 2,   // dW_x: A = x, B = dA, q a pulling position
  TN_DWXF = 3,  // dW_x[:, f]: A = x, B = dA_fk, q = k n_pull + pulling position
  TN_FC = 4,    // Tree-FC dW_k: A = h_k, B = delta
  TN_HEAD = 5,  // dW_s: A = h, B = dZ, q any position
};

struct X3Job {
  int kind, arg;               // arg: rows per slot (DUF, DWXF) or the slot (FC)
  int Q, qchunk, Mo, No, gap;  // B column n >= gap is H further (the skipped f block)
  int lda, ldb;                // elements per row index of A and of B
  int tx, ty, wg_end;
  const float *A, *B;
  float* out;
};
constexpr int kX3Jobs = 4;
struct X3Group {
  X3Job j[kX3Jobs];
  int n;
};

// block of a dA row that holds the forget gate of slot k (f_col / H)
__device__ __forceinline__ int f_blk(int k) { return k == 0 ? 1 : 3 + k; }

// rows of A and B (in units of J.lda and J.ldb) that are row q of the product
// (-1: a row of zeros).  The products with one block of dA count it in blocks
// of H.
__device__ __forceinline__ void x3_rows(const Net& n, const X3Job& J, int off1, int q, int& a,
                                        int& b) {
  switch (J.kind) {
    case TN_DU: {
      b = off1 + q;
      a = n.N == 1 ? n.child_pos[b] : b;
      return;
    }
    case TN_DUF: {
      const int k = q / J.arg, p = off1 + q - k * J.arg;
      a = n.child_pos[(size_t)p * n.N + k];
      b = p * (3 + n.N) + f_blk(k);
      return;
    }
    case TN_DWX: {
      b = n.pull_list[q];
      a = n.pull_pos[b];
      return;
    }
    case TN_DWXF: {
      const int k = q / J.arg, p = n.pull_list[q - k * J.arg];
      a = n.pull_pos[p];
      b = p * (3 + n.N) + f_blk(k);
      return;
    }
    case TN_FC: {
      b = off1 + q;
      a = n.child_pos[(size_t)b * n.N + J.arg];
      return;
    }
    default:
      a = b = q;
  }
}

// A 128 x 128 output tile per workgroup, wavefronts 2 x 2 of 64 x 64.
// Threads 0-127 load A, 128-255 B: thread (octet q, i) loads columns
// 4i .. 4i+3 of eight rows, 32 values, of the next chunk while this one is
// multiplied, then splits them into LDS (split3.h), transposed in registers.
// One 48 KB stage: three workgroups share a CU and cover each other's
// barriers, splits and loads.  The rows of a segment are looked up into LDS
// first; their 64-bit addresses are formed as they are loaded.  Against the fp32-instruction products it replaced
// (direct-to-LDS, 128 x 256 tiles, at 85-115 TFLOP/s): SST batch, dU, dU_f
// and dW_x (16.6 GFLOP) 177 -> 108 us in one launch instead of two; Tree-FC
// dW (17.1) 158 -> 98; chains (17.4) 135 -> 86; dW_s at 10 000 classes (23.3)
// 244 -> 145.  Without loads and splits it takes 70 us on Tree-FC, with a
// third of the fragment reads 64: the bf16 units themselves sustain about
// 1.7 PFLOP/s here.  Two workgroups a CU: 101.  Relative error of dU against
// 64 bits, before / after: Tree-FC 2.9e-6 / 2.8e-6, chains 6.6e-7 / 5.2e-7; dW_s
// at 10 000 classes 9.4e-7 / 5.1e-7.  On the SST batch, whose chains are the
// longest (22 chunks), 3.1e-7 / 3.3e-7 in one chain, 2.3e-7 with the chunks
// summed apart (104 -> 108 us): so above kX3Apart chunks, in the Tree-LSTM's
// products (chains: 19 chunks, 84 -> 86 us).
constexpr int kX3Seg = 512;
constexpr int kX3Apart = 18;

template <bool APART>
__global__ void __launch_bounds__(256, 3) k_x3_tn(Net n, int off1, X3Group G) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kX3Bytes];
  __shared__ __attribute__((aligned(16))) int rows[2][kX3Seg];
  const int item = xcd_item(blockIdx.x, G.j[G.n - 1].wg_end);
  if (item < 0) return;
  int jb = 0;
  while (jb + 1 < G.n && item >= G.j[jb].wg_end) ++jb;
  const X3Job& J = G.j[jb];
  const int wg = item - (jb > 0 ? G.j[jb - 1].wg_end : 0);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wm = w & 1, wn = w >> 1;
  const int m0 = wg % J.ty * kX3Tile, n0 = wg / J.ty % J.tx * kX3Tile, s = wg / (J.tx * J.ty);
  const int q_lo = s * J.qchunk, q_hi = min(J.Q, q_lo + J.qchunk);
  const int side = __builtin_amdgcn_readfirstlane(tid >> 7);
  char* const mine = lds + side * kX3Bytes;
  v4f acc[4][4];
  auto sum = [&](auto parts, int t, auto&& mma) {
    constexpr int P = decltype(parts)::value;
    const int oq = t >> 5, i = t & 31, col = (side ? n0 : m0) + 4 * i;
    const bool col_ok = col < (side ? J.No : J.Mo);
    const float* base = side ? J.B + col + (col >= J.gap ? n.H : 0) : J.A + col;
    const size_t ld = side ? J.ldb : J.lda;
    zero_acc(acc);
    for (int seg = q_lo; seg < q_hi; seg += kX3Seg) {
      const int nq = min(kX3Seg, q_hi - seg), nch = cdiv_dev(nq, kBK);
      __syncthreads();   // the previous segment's rows are consumed
      for (int x = tid; x < nch * kBK; x += 256) {
        int a = -1, b = -1;
        if (x < nq) x3_rows(n, J, off1, seg + x, a, b);
        rows[0][x] = a;
        rows[1][x] = a < 0 ? -1 : b;   // a zero row of A needs nothing of B
      }
      __syncthreads();
      float4 v[8];
      auto load = [&](int c) {
        const int4* o = reinterpret_cast<const int4*>(&rows[side][c * kBK + 8 * oq]);
        const int4 lo = o[0], hi = o[1];
        const int rv[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ldg4(col_ok && rv[e] >= 0 ? base + rv[e] * ld : n.zrow);
      };
      load(0);
      for (int c = 0; c < nch; ++c) {
        if (c > 0) __syncthreads();   // the previous chunk's fragments are read
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = j == 0 ? v[e].x : j == 1 ? v[e].y : j == 2 ? v[e].z : v[e].w;
          x3_store<P>(mine, 32 * j + i, oq, x);
        }
        __syncthreads();
        if (c + 1 < nch) load(c + 1);
        __builtin_amdgcn_sched_barrier(0);   // the next chunk's loads go out before these products
        mma();
      }
    }
  };
  sum(std::integral_constant<int, 3>{}, tid & 127,
      [&] { x3_mma<3, 15, APART>(lds, lds + kX3Bytes, wm, wn, acc); });
  if (x3_nan(acc))   // NaN, or an operand without parts (split3.h)
    sum(std::integral_constant<int, 0>{}, x3_again(tid & 127),
        [&] { x3_mma_f32(lds, lds + kX3Bytes, wm, wn, acc); });
  float* o = J.out + (size_t)s * J.Mo * J.No;
  const int nc = n0 + 64 * wn + 4 * r;
  if (nc >= J.No) return;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + 64 * wm + 16 * g + 4 * e + j;
      if (m < J.Mo)
        st4(o + (size_t)m * J.No + nc,
            make_float4(acc[j][0][e], acc[j][1][e], acc[j][2][e], acc[j][3][e]));
    }
}

// All pending split-K sums in one launch: blockIdx.y picks the job.  Kind 0:
// each thread adds four adjacent outputs with float4 access (every such
// job's No, ldd, col_off, gap_start and gap are multiples of 4, checked on
// the host).  Kind 1 (column sums with many partial rows): see below.
__global__ void __launch_bounds__(1024) k_reduce_jobs(SplitJobs jobs) {
  const SplitJob& J = jobs.j[blockIdx.y];
  if (J.kind == 1) {
    // 64 columns per block; wavefront y adds partial rows y, y + 16, ...,
    // then the 16 sums are added in order
    __shared__ float red[16][64];
    const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + x;
    if (blockIdx.x * 64 >= J.No) return;   // the whole block
    float t = 0.f;
    if (col < J.No)
      for (int k = y; k < J.S; k += 16) t += J.part[(size_t)k * J.No + col];
    red[y][x] = t;
    __syncthreads();
    if (y != 0 || col >= J.No) return;
    float u = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) u += red[k][x];
    J.dst[col] = u;
    return;
  }
  const long idx = 4 * ((long)blockIdx.x * 1024 + threadIdx.x);
  const long total = (long)J.Mo * J.No;
  if (idx >= total) return;
  const size_t stride = (size_t)total;
  const int m = (int)(idx / J.No), nn = (int)(idx % J.No);
  float4 s = f4zero();
#pragma unroll 4
  for (int k = 0; k < J.S; ++k) {
    const float4 v = ldg4(J.part + k * stride + idx);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  float* d = J.dst + (size_t)m * J.ldd + J.col_off + nn + (nn >= J.gap_start ? J.gap : 0);
  if (J.acc) {
    const float4 o = ldg4(d);
    s = make_float4(o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w);
  }
  st4(d, s);
}

// The reduction of a split-K product: queued on `jobs` when given (the
// caller then launches reduce_split_jobs), else launched at once.
void split_sum(const float* part, int S, int Mo, int No, float* dst, int ldd, int col_off,
               int gap_start, int gap, hipStream_t st, SplitJobs* jobs) {
  const bool by4 = No % 4 == 0 && ldd % 4 == 0 && col_off % 4 == 0 && gap % 4 == 0 &&
                   (gap_start % 4 == 0 || gap_start >= No) && (uintptr_t)dst % 16 == 0;
  if (jobs && jobs->n < SplitJobs::kMax && by4) {
    jobs->j[jobs->n++] = SplitJob{part, dst, S, Mo, No, ldd, col_off, gap_start, gap};
    return;
  }
  CAVS_LAUNCH("k_reduce_splits", k_reduce_splits, dim3(cdiv((long)Mo * No, 256)), dim3(256), 0, st,
              part, S, Mo, No, dst, ldd, col_off, gap_start, gap);
}

// ------------------------------------------- bf16 lazy products, packed
// With bf16 matrix-product operands a lazy product first packs both
// operands, rounded to bf16 (nearest-even) where the fp32 path would feed
// them to the matrix core, into rows that are contiguous in the contraction
// index q: pack row c < Mp is column m = c of A (zero for m >= Mo), row
// Mp + n is column n of B; every row holds Qp values (zero for q >= Q).  The
// product is then an "A B^T" over those rows, staged straight into LDS.
constexpr int kPackQ = kPackSeg;
constexpr int kNtTile = kPackTile;

template <class L>
__global__ void __launch_bounds__(256) k_pack_bf(L ld, int Q, int Qp, int Mo, int Mp,
                                                 u16* __restrict__ pk) {
  __shared__ u16 t[64][kPackQ + 8];   // [column][q]
  const int c0 = blockIdx.x * 64, q0 = blockIdx.y * kPackQ;
  const int tid = threadIdx.x, c4 = tid & 15, qr = tid >> 4;
  const bool aside = c0 < Mp;        // 64 | Mp: a block is all A or all B columns
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ql = qr + 16 * i, q = q0 + ql;
    float4 v = f4zero();
    if (q < Q) {
      const auto x = ld.idx(q);
      if (aside) {
        const int m = c0 + 4 * c4;
        if (m < Mo) v = ld.a4(x, q, m);
      } else {
        v = ld.b4(x, q, c0 - Mp + 4 * c4);
      }
    }
    t[4 * c4 + 0][ql] = f2bf(v.x);
    t[4 * c4 + 1][ql] = f2bf(v.y);
    t[4 * c4 + 2][ql] = f2bf(v.z);
    t[4 * c4 + 3][ql] = f2bf(v.w);
  }
  __syncthreads();
  // 64 columns x 64 q: thread (row, seg) writes 16 q (32 bytes) of one row
  const int row = tid >> 2, seg = tid & 3;
  const uint4* sp = reinterpret_cast<const uint4*>(&t[row][16 * seg]);
  uint4* dp = reinterpret_cast<uint4*>(pk + (size_t)(c0 + row) * Qp + q0 + 16 * seg);
  dp[0] = sp[0];
  dp[1] = sp[1];
}

// out[s][m][n] = sum over q in split s of pack[m][q] pack[Mp + n][q] for
// m < Mo: a 128 x 128 tile, four wavefronts of 64 x 64 (4 x 4 blocks of
// v_mfma_f32_16x16x32_bf16), 64-deep chunks through an S-stage ring of
// 128-byte LDS rows (quads XOR-swizzled by row & 7).  The n fragment is the
// MFMA's A operand, so lane (r, g) holds four consecutive n of one m.
__device__ __forceinline__ bf16x8 quad_sw(const float* L, int row, int q) {
  return *reinterpret_cast<const bf16x8*>(L + row * 32 + 4 * (q ^ (row & 7)));
}

template <int S>
__global__ void __launch_bounds__(256) k_nt_bf(const u16* __restrict__ pk, int Qp, int qchunk,
                                               int Mo, int Mp, int No, float* __restrict__ out) {
  constexpr int BM = kNtTile, BN = kNtTile, ROWS = BM + BN, IPW = ROWS / 32;
  __shared__ __attribute__((aligned(1024))) float L0[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L1[ROWS * 32];
  __shared__ __attribute__((aligned(1024))) float L2[S > 2 ? ROWS * 32 : 4];
  __shared__ __attribute__((aligned(1024))) float L3[S > 3 ? ROWS * 32 : 4];
  const Ring<ROWS, S> ring{L0, L1, L2, L3};
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wm = w & 1, wn = w >> 1;
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM, s = blockIdx.z;
  const int q_lo = s * qchunk, nch = (min(Qp, q_lo + qchunk) - q_lo) / kPackQ;
  // LDS rows [0, BM): pack rows m0 + row; [BM, ROWS): pack rows Mp + n0 + row - BM
  const char* src[IPW];
#pragma unroll
  for (int t = 0; t < IPW; ++t) {
    const int row = (w * IPW + t) * 8 + (lane >> 3), qg = (lane & 7) ^ (row & 7);
    const int prow = row < BM ? m0 + row : Mp + n0 + row - BM;
    src[t] = reinterpret_cast<const char*>(pk + (size_t)prow * Qp + q_lo) + 16 * qg;
  }
  const int wofs = __builtin_amdgcn_readfirstlane(w * IPW * 256);
  v4f acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
  auto issue = [&](auto sc, int c) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr_of(ring.at(sc)) + 4u * wofs);
#pragma unroll
    for (int t = 0; t < IPW; ++t)
      copy16_to_lds(reinterpret_cast<const float*>(src[t] + 128 * c), base + 1024u * t);
  };
  struct Frag {
    bf16x8 m[4][2], n[4][2];
  };
  auto read = [&](const float* Ls, Frag& f) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f.n[b][h] = quad_sw(Ls, BM + wn * 64 + b * 16 + r, 4 * h + g);
        f.m[b][h] = quad_sw(Ls, wm * 64 + b * 16 + r, 4 * h + g);
      }
  };
  auto mma = [&](const Frag& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma_bf16_16x16x32(f.n[b][h], f.m[a][h], acc[a][b]);
  };
  auto body = [&](const float* Lnext, Frag& cur, Frag& nxt, int) {
    read(Lnext, nxt);
    mma(cur);
    interleave_reads<16, 32>();
  };
  if (nch > 0) ring_loop_db<S, IPW, Frag>(nch, ring, issue, read, body);
  float* o = out + (size_t)s * Mo * No;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int m = m0 + wm * 64 + a * 16 + r;
    if (m >= Mo) continue;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      st4(o + (size_t)m * No + n0 + wn * 64 + b * 16 + 4 * g,
          make_float4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]));
  }
}

template <class L>
void tn_product(const L& ld, int Q, int Mo, int No, float* dst, int ldd, int col_off,
                int gap_start, int gap, float* part, size_t part_floats, hipStream_t st,
                SplitJobs* jobs = nullptr) {
  if (Q <= 0) {
    // empty contraction: zero output columns
    split_sum(part, 0, Mo, No, dst, ldd, col_off, gap_start, gap, st, jobs);
    return;
  }
  const Net& n = ld.n;
  // pack, then the packed product
  const int Mp = cdiv(Mo, kNtTile) * kNtTile, Qp = cdiv(Q, kPackQ) * kPackQ;
  if (n.pack && No % kNtTile == 0 && (size_t)(Mp + No) * Qp <= n.pack_elems) {
    CAVS_LAUNCH(L::kNamePack, k_pack_bf<L>, dim3((Mp + No) / 64, Qp / kPackQ), dim3(256), 0, st, ld,
                Q, Qp, Mo, Mp, n.pack);
    const int tiles = (No / kNtTile) * (Mp / kNtTile);
    int S = 256 / tiles;
    S = S < 1 ? 1 : S;
    if (S > Qp / kPackQ) S = Qp / kPackQ;
    while (S > 1 && (size_t)S * Mo * No > part_floats) --S;
    const int qchunk = cdiv(cdiv(Qp, S), kPackQ) * kPackQ;
    S = cdiv(Qp, qchunk);
    CAVS_LAUNCH(L::kNameNt, k_nt_bf<3>, dim3(No / kNtTile, Mp / kNtTile, S), dim3(256), 0, st,
                n.pack, Qp, qchunk, Mo, Mp, No, part);
    split_sum(part, S, Mo, No, dst, ldd, col_off, gap_start, gap, st, jobs);
    return;
  }
  const int tiles = (No / 64) * cdiv(Mo, 64);
  // about two workgroups per CU (256 CUs), never three on some: a CU's
  // co-resident workgroups share its matrix cores, so the busiest CU sets
  // the time
  int S = 512 / tiles;
  S = S < 1 ? 1 : S;
  S = S > kSplitCap ? kSplitCap : S;
  int maxS = cdiv(Q, 256);
  if (S > maxS) S = maxS;
  while (S > 1 && (size_t)S * Mo * No > part_floats) --S;
  int qchunk = cdiv(cdiv(Q, S), kBK) * kBK;
  S = cdiv(Q, qchunk);
  CAVS_LAUNCH(L::kNameBf, k_tn_gemm_bf<L>, dim3(No / 64, cdiv(Mo, 64), S), dim3(256), 0, st, ld, Q,
              qchunk, Mo, No, part);
  split_sum(part, S, Mo, No, dst, ldd, col_off, gap_start, gap, st, jobs);
}

// -------------------------------------------------------------- col sums
// The bias and head gradients are column sums over the level-major rows
// (lazy batching, Section 3.4): db sums dA (LSTM: 4H columns with
// f = f_0 + f_1; FC: H columns) over rows [row0, row1); dW_s[j][c] sums
// h_j dZ_c and db_s[c] sums dZ_c over all rows.  One launch writes per-chunk
// partials (each thread: 4 adjacent columns, its chunk's rows in order); the
// split-K reduction launch adds the chunks in order, so the result is
// deterministic.
constexpr int kBiasChunks = 256;

// Partial sums of chunk y: db columns at part[y * wA + c], dW_s at
// part[nchunk * wA + y * H C + j C + c], db_s at
// part[nchunk * (wA + H C) + y C + c]: three arrays whose chunk-major rows
// are each one split-K reduction job.
template <int CP4>
__global__ void __launch_bounds__(256) k_bias_part(Net n, int row0, int row1, int lo1,
                                                   int rows_per, int bxA, int wA, int nchunk,
                                                   float* __restrict__ part) {
  const int H = n.H;
  const int lo = blockIdx.y * rows_per, hi = min(n.V, lo + rows_per);
  if ((int)blockIdx.x < bxA) {
    const int c = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (c >= wA) return;
    int r0 = max(lo, row0);
    const int r1 = min(hi, row1);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (n.GW == H) {  // Tree-FC
#pragma unroll 4
      for (int p = r0; p < r1; ++p) {
        const float4 v = *reinterpret_cast<const float4*>(n.dA + (size_t)p * H + c);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
    } else {
      const bool fcol = c >= G_F * H && c < (G_F + 1) * H;
      if (fcol) r0 = max(r0, lo1);  // level-0 rows have no children: f is zero
      const int nf = fcol ? n.N : 1;   // forget blocks that make up the column
#pragma unroll 4
      for (int p = r0; p < r1; ++p) {
        const float* row = n.dA + (size_t)p * n.GW;
        float4 v = *reinterpret_cast<const float4*>(row + c);
        for (int k = 1; k < nf; ++k) {
          const float4 u = *reinterpret_cast<const float4*>(row + (2 + k) * H + c);
          v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
    }
    *reinterpret_cast<float4*>(part + (size_t)blockIdx.y * wA + c) = s;
    return;
  }
  // head: columns wA + j*C + c (dW_s row-major), then wA + H*C + c (db_s);
  // dZ rows hold CP = 4 CP4 columns, zero past C
  const int j = 4 * ((blockIdx.x - bxA) * 256 + threadIdx.x);
  if (j >= H) return;
  const int C = n.C;
  constexpr int CP = 4 * CP4;
  float acc[4][CP], zs[CP];
#pragma unroll
  for (int c = 0; c < CP; ++c) {
    zs[c] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e][c] = 0.f;
  }
#pragma unroll 4
  for (int p = lo; p < hi; ++p) {
    const float4 h = *reinterpret_cast<const float4*>(n.Hs + (size_t)p * H + j);
    const float4* dz = reinterpret_cast<const float4*>(n.dZ + (size_t)p * CP);
#pragma unroll
    for (int c4 = 0; c4 < CP4; ++c4) {
      const float4 z4 = dz[c4];
      const float z[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * c4 + e;
        acc[0][c] += h.x * z[e];
        acc[1][c] += h.y * z[e];
        acc[2][c] += h.z * z[e];
        acc[3][c] += h.w * z[e];
        zs[c] += z[e];
      }
    }
  }
  const size_t HC = (size_t)H * C;
  float* o = part + (size_t)nchunk * wA + blockIdx.y * HC + (size_t)j * C;
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int c = 0; c < CP; ++c)
      if (c < C) o[e * C + c] = acc[e][c];
  if (j == 0) {
    float* ob = part + (size_t)nchunk * (wA + HC) + (size_t)blockIdx.y * C;
#pragma unroll
    for (int c = 0; c < CP; ++c)
      if (c < C) ob[c] = zs[c];
  }
}

// ---------------------------------------------------------------- loss
// Cross-entropy head over every position (the push of Section 3.4, batched
// lazily).  A workgroup owns 16 positions; its eight wavefronts split both
// products:
//   z = h W_s + b_s       16 positions x 16 class columns on MFMA, wavefront
//                         w taking the K chunks w, w+8, ... (MC at a time,
//                         loads first); the eight partial blocks are added in
//                         order in LDS (columns >= C repeat class C-1 and are
//                         masked);
//   log-sum-exp and softmax across the 16 lanes that hold a row's classes;
//   dZ = (softmax - onehot(label)) / |Lambda| for labelled positions, zero
//   rows otherwise (row stride CP, pad columns zero);
//   dHL = dZ W_s^T, the head's share of dL/dh, on MFMA (K = CP), wavefront w
//   taking the 16-unit blocks w, w+8, ...
// Inference (dZ and dHL null) stops after the per-position loss terms.
constexpr int kLossWaves = 8;

template <int MC>
__global__ void __launch_bounds__(64 * kLossWaves) k_loss_ce(Net n) {
  constexpr int NW = kLossWaves;
  __shared__ float zp[NW][16][17];
  __shared__ float dzl[16][17];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int p0 = blockIdx.x * 16;
  const int H = n.H, C = n.C, CP = n.CP, V = n.V;
  if (blockIdx.x == 0)   // the zero row the lazy products read for absent rows
    for (int j = threadIdx.x; j < H; j += 64 * kLossWaves) n.zrow[j] = 0.f;
  const int cm = min(r, C - 1);
  const bool cval = r < C;
  // loads unconditional (rows past V read row V-1, masked below), so that
  // they issue together
  int q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = n.push_pos[min(p0 + 4 * g + i, V - 1)];
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = p0 + 4 * g + i < V ? q[i] : -1;
  const float bsc = n.bs[cm];

  const float* hrow = n.Hs + (size_t)min(p0 + r, V - 1) * H + 8 * g;
  const float* wcol = n.Ws + cm;
  const int nch = H / kBK;
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = w; c0 < nch; c0 += NW * MC) {
    float a[MC][8], b[MC][8];
#pragma unroll
    for (int t = 0; t < MC; ++t) {
      const int k0 = min(c0 + NW * t, nch - 1) * kBK;
      ld8(hrow + k0, a[t]);
#pragma unroll
      for (int s2 = 0; s2 < 8; ++s2) b[t][s2] = wcol[(size_t)(k0 + 8 * g + s2) * C];
    }
#pragma unroll
    for (int t = 0; t < MC; ++t)
      if (c0 + NW * t < nch) acc = mfma_chunk8<false>(a[t], b[t], acc);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) zp[w][4 * g + i][r] = acc[i];
  __syncthreads();

  // wavefront i < 4 finishes row i of each lane group (16 lanes per row,
  // one class per lane)
  if (w < 4) {
    const int i = w;
    const int p = p0 + 4 * g + i;
    float z = zp[0][4 * g + i][r];
#pragma unroll
    for (int v = 1; v < NW; ++v) z += zp[v][4 * g + i][r];
    z += bsc;
    // log-sum-exp and softmax of the logits in fp64 (C exponentials per
    // vertex, a negligible cost): with small logits every vertex computes
    // nearly the same lse, so an fp32 rounding of it would repeat in every
    // row of dZ and add up coherently in the sums over vertices (db, db_s)
    const double zd = (double)z;
    double m = cval ? zd : -INFINITY;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, kWave));
    double se = cval ? exp(zd - m) : 0.0;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) se += __shfl_xor(se, o, kWave);
    const double lse = m + log(se);
    float d = 0.f;
    if (q[i] >= 0 && cval)
      d = (float)((exp(zd - lse) - (r == q[i] ? 1.0 : 0.0)) * (double)n.inv_denom);
    dzl[4 * g + i][r] = d;
    if (p < V) {
      if (r < CP && n.dZ) n.dZ[(size_t)p * CP + r] = d;
      if (q[i] < 0 && r == 0) n.lossv[p] = 0.f;
      if (q[i] >= 0 && r == q[i]) n.lossv[p] = (float)(lse - zd);
    }
  }
  if (!n.dHL) return;   // inference: no gradient of the head
  __syncthreads();
  float a[4];
  const int KT = CP / 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = t < KT ? dzl[r][4 * t + g] : 0.f;
  const int nb = H / 16;
  constexpr int MB = 4;
  for (int b0 = w; b0 < nb; b0 += NW * MB) {
    float wb[MB][4];
#pragma unroll
    for (int u = 0; u < MB; ++u) {
      const float* wrow = n.Ws + (size_t)(min(b0 + NW * u, nb - 1) * 16 + r) * C;
#pragma unroll
      for (int t = 0; t < 4; ++t) wb[u][t] = wrow[min(4 * t + g, C - 1)];
    }
    // classes past CP are never multiplied (t < KT below)
#pragma unroll
    for (int u = 0; u < MB; ++u) {
      const int jb = b0 + NW * u;
      if (jb >= nb) break;
      v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (t < KT) o = mfma_f32_16x16x4(a[t], wb[u][t], o);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = p0 + 4 * g + i;
        if (p < V) n.dHL[(size_t)p * H + jb * 16 + r] = o[i];
      }
    }
  }
}

// Squared-error head: one wavefront per position; loss 0.5 |h - y|^2 and
// dHL = (h - y) / |Lambda| (zero rows for unlabelled positions; not written
// in inference, where dHL is null).
__global__ void __launch_bounds__(256) k_loss_l2(Net n) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int p = blockIdx.x * 4 + w;
  if (blockIdx.x == 0)   // the zero row the lazy products read for absent rows
    for (int j = threadIdx.x; j < n.H; j += 256) n.zrow[j] = 0.f;
  if (p >= n.V) return;
  const int q = n.push_pos[p], H = n.H;
  const float* h = n.Hs + (size_t)p * H;
  float* dh = n.dHL ? n.dHL + (size_t)p * H : nullptr;   // null in inference
  if (q < 0) {
    if (lane == 0) n.lossv[p] = 0.f;
    if (dh)
      for (int j = lane; j < H; j += 64) dh[j] = 0.f;
    return;
  }
  const float* y = n.Y + (size_t)q * H;
  float s = 0.f;
  for (int j = lane; j < H; j += 64) {
    const float d = h[j] - y[j];
    s += d * d;
    if (dh) dh[j] = d * n.inv_denom;
  }
  s = wave_sum(s);
  if (lane == 0) n.lossv[p] = 0.5f * s;
}

__global__ void __launch_bounds__(1024) k_loss_sum(const float* __restrict__ lossv, int V,
                                                   float scale, float* out) {
  __shared__ float red[1024];
  float s = 0.f;
  for (int i = threadIdx.x; i < V; i += 1024) s += lossv[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 512; o >= 1; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0] * scale;
}

}  // namespace

size_t lazy_part_floats(int V, int D, int H, int N, int C) {
  (void)V;
  size_t a = (size_t)kMaxSplits * 4 * H * (size_t)H;        // dU / FC dW
  size_t b = (size_t)kMaxSplits * 4 * H * (size_t)(D + 64);  // dW_x (m tail padding)
  size_t c = (size_t)kBiasChunks * (4 * H + (size_t)(H + 1) * (C > 0 ? C : 0));
  (void)N;
  size_t m = a > b ? a : b;
  return m > c ? m : c;
}

void pull_gemm(const Net& n, int n_pull, bool with_f, int lo1, hipStream_t s) {
  if (n_pull <= 0) return;
  if (x3_pull_applies(n, n_pull)) {
    pull_gemm_x3(n, n_pull, with_f, lo1, s);
    return;
  }
  const dim3 grid(cdiv(n_pull, 64) * (n.H / 32));
  if (with_f)
    CAVS_LAUNCH("k_pull_tile<4, 64, 2>", (k_pull_tile<4, 64, 2>), grid, dim3(256), 0, s, n,
                n_pull, lo1);
  else
    CAVS_LAUNCH("k_pull_tile<3, 64, 2>", (k_pull_tile<3, 64, 2>), grid, dim3(256), 0, s, n,
                n_pull, lo1);
}

void dx_gemm(const Net& n, int n_pull, bool with_f, float* dX, hipStream_t s) {
  if (n_pull <= 0) return;
  if (n.bf) {
    const dim3 g64(cdiv(n_pull, 64), cdiv(n.D, 64));
    if (g64.x * g64.y <= 1024)   // one round, four to a CU
      CAVS_LAUNCH("k_dx_gemm_bf", k_dx_gemm_bf, g64, dim3(256), 0, s, n, n_pull, (int)with_f, dX);
    else
      dx_gemm_bf(n, n_pull, with_f, dX, s);
    return;
  }
  // 32-row tiles: about three workgroups per CU at the benchmark shapes
  const dim3 grid(cdiv(n_pull, 32), cdiv(n.D, 64));
  if (with_f && n.N > 1)
    CAVS_LAUNCH("k_dx_tile<32, 64, 3, slots>", (k_dx_tile<32, 64, 3, true>), grid, dim3(256), 0, s,
                n, n_pull, (int)with_f, dX);
  else
    CAVS_LAUNCH("k_dx_tile<32, 64, 3>", (k_dx_tile<32, 64, 3, false>), grid, dim3(256), 0, s, n,
                n_pull, (int)with_f, dX);
}

// dhlx[p] = dHL[p] + ext[vertex of p]: the gradient an external consumer of
// the pushed states sends back (vertex-id rows), joined to the loss head's.
__global__ void __launch_bounds__(256) k_add_ext(Net n, const float* __restrict__ ext,
                                                 float* __restrict__ dhlx) {
  const int q = n.H / 4;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)n.V * q) return;
  const int p = (int)(i / q), j0 = 4 * (int)(i % q);
  const int v = n.order[p];
  st4(dhlx + (size_t)p * n.H + j0,
      add4(ldg4(n.dHL + (size_t)p * n.H + j0), ldg4(ext + (size_t)v * n.H + j0)));
}

void add_external_grad(const Net& n, const float* ext, float* dhlx, hipStream_t s) {
  if (n.V <= 0) return;
  CAVS_LAUNCH("k_add_ext", k_add_ext, dim3(cdiv((long)n.V * (n.H / 4), 256)), dim3(256), 0, s, n,
              ext, dhlx);
}

void loss_fwd(const Net& n, float* loss_out, float* part, size_t part_cap, hipStream_t s) {
  if (n.loss == CAVS_LOSS_NONE || (n.loss == CAVS_LOSS_CE && n.C > kSmallHeadC))
    (void)zero_async(n.zrow, (size_t)n.H * sizeof(float), s);   // the small heads' kernels clear it
  if (n.loss == CAVS_LOSS_NONE) {   // states pushed to an external consumer only
    (void)zero_async(n.lossv, (size_t)n.V * sizeof(float), s);
    if (n.dHL) (void)zero_async(n.dHL, (size_t)n.V * n.H * sizeof(float), s);
  } else if (n.loss == CAVS_LOSS_CE && n.C > kSmallHeadC) {
    lm_head_fwd(n, part, part_cap, s);
  } else if (n.loss == CAVS_LOSS_CE) {
    const int per = cdiv(n.H / kBK, kLossWaves);  // K chunks per wavefront
    const dim3 grid(cdiv(n.V, 16)), block(64 * kLossWaves);
    if (per <= 1) CAVS_LAUNCH("k_loss_ce<1>", k_loss_ce<1>, grid, block, 0, s, n);
    else if (per <= 2) CAVS_LAUNCH("k_loss_ce<2>", k_loss_ce<2>, grid, block, 0, s, n);
    else CAVS_LAUNCH("k_loss_ce<4>", k_loss_ce<4>, grid, block, 0, s, n);
  } else {
    CAVS_LAUNCH("k_loss_l2", k_loss_l2, dim3(cdiv(n.V, 4)), dim3(256), 0, s, n);
  }
  CAVS_LAUNCH("k_loss_sum", k_loss_sum, dim3(1), dim3(1024), 0, s, (const float*)n.lossv, n.V,
                     n.inv_denom, loss_out);
}

// One lazy product of an fp32 pass: the job, where its sum goes (as in
// split_sum) and its scratch.
struct X3Plan {
  X3Job job;
  float* dst;
  int ldd, col_off;
  float* part;
  size_t part_floats;
  bool direct;   // an unsplit product may write dst itself
};

// At most this many workgroups: one round, three per CU.
constexpr int kX3WGs = 768;

// All products of a pass in one grid.  Split counts: the fewest 32-deep
// chunks per workgroup for which every product, split so that no workgroup
// carries more, fits the launch in one round; one chunk each only up to a
// workgroup per CU.  us, product and sum of its splits, one chunk / two: Tree-FC
// dW, H = 256, 32 workgroups 6 + 4 / 8 + 4, 496 (62 splits) 11 + 12 / 11 + 7;
// H = 1024, 512 workgroups 11.4 + 6.7 / 10.8 + 5.2.
void x3_tn_launch(const char* name, const Net& n, int off1, X3Plan* P, int np, hipStream_t st,
                  SplitJobs* jobs) {
  int nch[kX3Jobs], tiles[kX3Jobs], cap[kX3Jobs], most = 1;
  for (int k = 0; k < np; ++k) {
    const X3Job& J = P[k].job;
    nch[k] = cdiv(J.Q, kBK);
    tiles[k] = cdiv(J.No, kX3Tile) * cdiv(J.Mo, kX3Tile);
    const size_t fit = P[k].part_floats / ((size_t)J.Mo * J.No);
    cap[k] = (int)std::min<size_t>(fit > 0 ? fit : 1, (size_t)std::max(nch[k], 1));
    most = std::max(most, nch[k]);
  }
  auto splits = [&](int k, int per) { return std::min(cap[k], cdiv(nch[k], per)); };
  auto wgs = [&](int per) {
    long t = 0;
    for (int k = 0; k < np; ++k) t += (long)tiles[k] * splits(k, per);
    return t;
  };
  // wgs() does not increase with the chunks per workgroup
  int lo = wgs(1) <= 256 ? 1 : 2, hi = std::max(most, lo);
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (wgs(mid) <= kX3WGs) hi = mid;
    else lo = mid + 1;
  }
  X3Group G{};
  int end = 0, S[kX3Jobs];
  for (int k = 0; k < np; ++k) {
    X3Job& J = P[k].job;
    S[k] = 0;
    if (nch[k] == 0) continue;
    J.qchunk = cdiv(nch[k], splits(k, lo)) * kBK;
    S[k] = cdiv(J.Q, J.qchunk);
    J.tx = cdiv(J.No, kX3Tile);
    J.ty = cdiv(J.Mo, kX3Tile);
    end += J.tx * J.ty * S[k];
    J.wg_end = end;
    // one split of a product that fills its destination's rows is the result
    J.out = P[k].direct && S[k] == 1 && P[k].ldd == J.No && (uintptr_t)P[k].dst % 16 == 0
                ? P[k].dst
                : P[k].part;
    G.j[G.n++] = J;
  }
  if (end > 0 && lo > kX3Apart && P[0].job.kind < TN_FC)
    CAVS_LAUNCH(name, k_x3_tn<true>, dim3(xcd_grid(end)), dim3(256), 0, st, n, off1, G);
  else if (end > 0)
    CAVS_LAUNCH(name, k_x3_tn<false>, dim3(xcd_grid(end)), dim3(256), 0, st, n, off1, G);
  for (int k = 0; k < np; ++k) {
    const X3Job& J = P[k].job;
    if (nch[k] > 0 && J.out == P[k].dst) continue;
    const bool gap = J.gap < J.No;
    split_sum(P[k].part, S[k], J.Mo, J.No, P[k].dst, P[k].ldd, P[k].col_off,
              gap ? J.gap : 1 << 30, gap ? n.H : 0, st, jobs);
  }
}

constexpr int kNoGap = 1 << 30;
X3Plan x3_plan(int kind, int arg, int Q, int Mo, int No, int gap, const float* A, int lda,
               const float* B, int ldb, float* dst, int ldd, int col_off, float* part, size_t pf) {
  X3Job J{};
  J.kind = kind;
  J.arg = arg;
  J.Q = Q;
  J.Mo = Mo;
  J.No = No;
  J.gap = gap;
  J.A = A;
  J.B = B;
  J.lda = lda;
  J.ldb = ldb;
  return X3Plan{J, dst, ldd, col_off, part, pf, true};
}

// dW_x scratch: three quarters of a product's share for i|o|u, the rest for
// the f columns where they are a product of their own
size_t dwx_iou_floats(size_t pf) { return pf / 4 * 3; }

X3Plan plan_dU(const Net& n, int MI, float* dU, float* part, size_t pf) {
  const int H = n.H;
  if (n.N == 1)
    return x3_plan(TN_DU, 0, MI, H, 4 * H, kNoGap, n.Hs, H, n.dA, n.GW, dU, 4 * H, 0, part, pf);
  return x3_plan(TN_DU, 0, MI, H, 3 * H, H, n.Ht, H, n.dA, n.GW, dU, 4 * H, 0, part, pf);
}
X3Plan plan_dUf(const Net& n, int MI, float* dU, float* part, size_t pf) {
  const int H = n.H;
  return x3_plan(TN_DUF, MI, n.N * MI, H, H, kNoGap, n.Hs, H, n.dA, H, dU, 4 * H, H, part, pf);
}
// the product(s) of dW_x; returns how many
int plan_dWx(const Net& n, int n_pull, bool with_f, float* dWx, float* part, size_t pf,
             X3Plan* P) {
  const int H = n.H, D = n.D;
  if (with_f && n.N == 1) {
    P[0] = x3_plan(TN_DWX, 0, n_pull, D, 4 * H, kNoGap, n.X, D, n.dA, n.GW, dWx, 4 * H, 0, part, pf);
    return 1;
  }
  const size_t px = dwx_iou_floats(pf);
  P[0] = x3_plan(TN_DWX, 0, n_pull, D, 3 * H, H, n.X, D, n.dA, n.GW, dWx, 4 * H, 0, part, px);
  if (!with_f) return 1;
  P[1] = x3_plan(TN_DWXF, n_pull, n.N * n_pull, D, H, kNoGap, n.X, D, n.dA, H, dWx, 4 * H, H,
                 part + px, pf - px);
  return 2;
}

bool lstm_lazy_grouped(const Net& n, int off1, int n_pull, bool with_f, float* dU, float* dWx,
                       float* part, size_t pf, hipStream_t s, SplitJobs* jobs) {
  const int H = n.H, D = n.D, MI = n.V - off1;
  if (n.bf) return false;
  X3Plan P[kX3Jobs];
  int np = 0;
  P[np++] = plan_dU(n, MI, dU, part, pf);
  if (n.N > 1) P[np++] = plan_dUf(n, MI, dU, part + pf, pf);
  if (D > 0) np += plan_dWx(n, n_pull, with_f, dWx, part + 2 * pf, pf, P + np);
  x3_tn_launch("k_x3_tn<lstm>", n, off1, P, np, s, jobs);
  // the f block of dW_x is exactly zero when no vertex with children pulls
  if (D > 0 && !with_f) split_sum(part + 2 * pf, 0, D, H, dWx, 4 * H, H, 1 << 30, 0, s, jobs);
  return true;
}

void lstm_dU_iou(const Net& n, int off1, float* dU, float* part, size_t part_floats,
                 hipStream_t s, SplitJobs* jobs, int rows) {
  const int H = n.H, MI = rows >= 0 ? rows : n.V - off1;
  if (!n.bf) {
    X3Plan P = plan_dU(n, MI, dU, part, part_floats);
    P.direct = rows < 0;   // a level's share is added to dU by its reduction
    x3_tn_launch("k_x3_tn<dU>", n, off1, &P, 1, s, jobs);
    return;
  }
  const LdDUiou ld{n, off1};
  if (n.N == 1) tn_product(ld, MI, H, 4 * H, dU, 4 * H, 0, 1 << 30, 0, part, part_floats, s, jobs);
  else tn_product(ld, MI, H, 3 * H, dU, 4 * H, 0, H, H, part, part_floats, s, jobs);
}

void lstm_dU_f(const Net& n, int off1, float* dU, float* part, size_t part_floats, hipStream_t s,
               SplitJobs* jobs, int rows) {
  if (n.N < 2) return;
  const int H = n.H, MI = rows >= 0 ? rows : n.V - off1;
  if (!n.bf) {
    X3Plan P = plan_dUf(n, MI, dU, part, part_floats);
    P.direct = rows < 0;
    x3_tn_launch("k_x3_tn<dUf>", n, off1, &P, 1, s, jobs);
    return;
  }
  LdDUf lf{n, off1, MI};
  tn_product(lf, n.N * MI, H, H, dU, 4 * H, H, 1 << 30, 0, part, part_floats, s, jobs);
}

void reduce_split_jobs(const SplitJobs& jobs, hipStream_t s) {
  if (jobs.n == 0) return;
  long most = 0;
  for (int k = 0; k < jobs.n; ++k) {
    const SplitJob& J = jobs.j[k];
    // elements per block: 4096 (four per thread), or 64 columns of a kind-1 job
    const long e = J.kind == 1 ? (long)cdiv(J.No, 64) * 4096 : (long)J.Mo * J.No;
    most = e > most ? e : most;
  }
  CAVS_LAUNCH("k_reduce_jobs", k_reduce_jobs, dim3(cdiv(most, 4096), jobs.n), dim3(1024), 0, s,
              jobs);
}

void lstm_dWx(const Net& n, int n_pull, bool with_f, float* dWx, float* part,
              size_t part_floats, hipStream_t s, SplitJobs* jobs) {
  const int H = n.H;
  if (!n.bf) {
    X3Plan P[2];
    const int np = plan_dWx(n, n_pull, with_f, dWx, part, part_floats, P);
    x3_tn_launch("k_x3_tn<dWx>", n, 0, P, np, s, jobs);
  } else if (with_f) {
    tn_product(LdDWx{n, 1}, n_pull, n.D, 4 * H, dWx, 4 * H, 0, 1 << 30, 0, part, part_floats, s,
               jobs);
  } else {
    tn_product(LdDWx{n, 0}, n_pull, n.D, 3 * H, dWx, 4 * H, 0, H, H, part, part_floats, s, jobs);
  }
  if (!with_f)   // the f block of dW_x is exactly zero: no vertex with children pulls
    split_sum(part, 0, n.D, H, dWx, 4 * H, H, 1 << 30, 0, s, jobs);
}

void fc_dW(const Net& n, int off1, float* dW, float* part, size_t part_floats, hipStream_t s,
           SplitJobs* jobs) {
  const int H = n.H, MI = n.V - off1;
  // the child slots' products share one launch; their split-K partials sit
  // side by side
  X3Plan P[kX3Jobs];
  for (int k = 0; k < n.N; ++k)
    P[k] = x3_plan(TN_FC, k, MI, H, H, kNoGap, n.Hs, H, n.dA, H, dW + (size_t)k * H * H, H, 0,
                   part + k * part_floats, part_floats);
  x3_tn_launch("k_x3_tn<FCdW>", n, off1, P, n.N, s, jobs);
}

void lm_dWs(const Net& n, float* dWs, float* part, size_t part_floats, hipStream_t s) {
  X3Plan P = x3_plan(TN_HEAD, 0, n.V, n.H, n.C, kNoGap, n.Hs, n.H, n.dZ, n.CP, dWs, n.C, 0, part,
                     part_floats);
  SplitJobs jobs;
  x3_tn_launch("k_x3_tn<lm_dWs>", n, 0, &P, 1, s, &jobs);
  reduce_split_jobs(jobs, s);
}

size_t bias_part_floats(int H, int C) {
  return (size_t)kBiasChunks * (4 * (size_t)H + (size_t)H * (C > 0 ? C : 0) + (C > 0 ? C : 0));
}

void bias_head_grads(const Net& n, int row0, int row1, int lo1, float* db, float* dWs, float* dbs,
                     float* part, hipStream_t s, SplitJobs* jobs) {
  const int wA = n.GW == n.H ? n.H : 4 * n.H;
  const bool head = n.loss == CAVS_LOSS_CE && n.C <= kSmallHeadC;   // the LM head has its own
  const int HC = head ? n.H * n.C : 0;
  int nchunk = cdiv(n.V, 16);
  if (nchunk > kBiasChunks) nchunk = kBiasChunks;
  if (nchunk < 1) nchunk = 1;
  const int rows_per = cdiv(n.V > 0 ? n.V : 1, nchunk);
  nchunk = cdiv(n.V > 0 ? n.V : 1, rows_per);
  const int bxA = cdiv(wA / 4, 256), bxB = head ? cdiv(n.H / 4, 256) : 0;
  const dim3 grid(bxA + bxB, nchunk);
  auto part_launch = [&](auto kern, const char* name) {
    CAVS_LAUNCH(name, kern, grid, dim3(256), 0, s, n, row0, row1, lo1, rows_per, bxA, wA, nchunk,
                part);
  };
  switch (head ? n.CP / 4 : 1) {
    case 1: part_launch(k_bias_part<1>, "k_bias_part<1>"); break;
    case 2: part_launch(k_bias_part<2>, "k_bias_part<2>"); break;
    case 3: part_launch(k_bias_part<3>, "k_bias_part<3>"); break;
    default: part_launch(k_bias_part<4>, "k_bias_part<4>"); break;
  }
  auto queue = [&](const float* p, int No, float* dst) {
    jobs->j[jobs->n++] = SplitJob{p, dst, nchunk, 1, No, No, 0, 1 << 30, 0, 1};
  };
  queue(part, wA, db);
  if (head) {
    queue(part + (size_t)nchunk * wA, HC, dWs);
    queue(part + (size_t)nchunk * (wA + HC), n.C, dbs);
  }
}

}  // namespace cavs

// Child-sum Tree-LSTM vertex function F and its gradient dF, one batching
// task (level) per launch (Algorithm 1; F as in the Tree-LSTM figure of
// Section 3.1).
//
// Forward, level t >= 1 (every vertex has a child): one kernel gathers the
// children's h rows straight from the level-major state buffer into LDS (the
// gather of Algorithm 2 fused into the operand load), forms h~ = h_0 + h_1 in
// registers, runs the five products h~ U_i, h~ U_o, h~ U_u, h_0 U_f, h_1 U_f
// on the matrix cores, and applies the gates, the cell update and the scatter
// of (c, h) in the epilogue (the elementwise fusion of Section 3.5).  The
// pulled-input term x W_x was produced beforehand by one GEMM over all
// vertices (pull is eager).  Level 0 (leaves) is elementwise.
//
// Backward, reverse level order: one GEMM kernel per level computes
// dL/dh_k = dA_iou U_iou^T + dA_fk U_f^T for every child k.  A vertex has one
// parent, so that product is the child's whole dL/dh: the epilogue turns it
// (with the dL/dc scattered earlier and the child's own loss term) into the
// child's pre-activation gradients dA, kept level-major for the lazy weight
// gradients, and scatters dL/dc_k' = g_c * f_k' to the grandchildren.  Roots
// are handled by one kernel before the level loop.  Every child row is
// written by exactly one thread: plain stores, no atomics.
#include <stdlib.h>

#include <map>

#include "lstm_dev.h"

namespace cavs {
namespace {

// ------------------------------------------------------------------ forward
__global__ void __launch_bounds__(256) k_lstm_leaf(Net n, int off, int M) {
  const int H = n.H;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)M * H) return;
  const int p = off + (int)(idx / H), j = (int)(idx % H);
  if (n.pull_pos[p] >= 0) return;   // finished by the pull product
  const float ai = n.b[G_I * H + j], ao = n.b[G_O * H + j], au = n.b[G_U * H + j];
  const float i = sigmoidf_(ai), o = sigmoidf_(ao), u = tanh_(au);
  const float c = i * u, h = o * tanh_(c);
  n.Hs[(size_t)p * H + j] = h;
  n.Cs[(size_t)p * H + j] = c;
  // a leaf has no forget gates: their saved columns are never read
  if (n.Gs) {   // null in inference
    float* g = n.Gs + (size_t)p * n.GW;
    g[j] = i;
    g[2 * H + j] = o;
    g[3 * H + j] = u;
  }
  const int v = n.order[p];
  n.h_out[(size_t)v * H + j] = h;
  if (n.c_out) n.c_out[(size_t)v * H + j] = c;
}

// dA of every position of a level below n.fuse_from (dL/dh, dL/dc stored by
// the parent; zero at a root), four consecutive units per thread with
// 16-byte accesses; with wb also its bf16 copy dAb (the operand rows of the
// bf16 backward product, rounded as that product rounds them).  LEAF:
// the level is the leaves (no children).  Loads are unconditional (a root's
// parent terms and an absent child's state read stale rows, masked by
// selects), and each element's arithmetic is that of lstm_gates_fin.
template <int NCH, bool LEAF>
__global__ void __launch_bounds__(256) k_lstm_bwd_gates4(Net n, int off, int M, int wb) {
  const int H = n.H, Hq = H / 4;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)M * Hq) return;
  const int p = off + (int)(idx / Hq), j0 = 4 * (int)(idx % Hq);
  const size_t row = (size_t)p * H + j0;
  const bool root = n.parent_pos[p] < 0;
  const float* g = n.Gs + (size_t)p * n.GW + j0;
  const float4 ig4 = ldg4(g), og4 = ldg4(g + 2 * H), ug4 = ldg4(g + 3 * H);
  const float4 c4 = ldg4(n.Cs + row), lg4 = ldg4(n.dHL + row);
  const float4 gh4 = ldg4(n.dHp + row), gi4 = ldg4(n.dCp + row);
  int cp[NCH];
  float4 fk4[NCH], ck4[NCH];
  if constexpr (!LEAF) {
#pragma unroll
    for (int k = 0; k < NCH; ++k) cp[k] = n.child_pos[(size_t)p * NCH + k];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      fk4[k] = ldg4(g + f_col(k, H));
      ck4[k] = ldg4(n.Cs + (size_t)max(cp[k], 0) * H + j0);
    }
  }
  const float ig[4] = {ig4.x, ig4.y, ig4.z, ig4.w}, og[4] = {og4.x, og4.y, og4.z, og4.w};
  const float ug[4] = {ug4.x, ug4.y, ug4.z, ug4.w}, cc[4] = {c4.x, c4.y, c4.z, c4.w};
  const float lg[4] = {lg4.x, lg4.y, lg4.z, lg4.w};
  const float ghp[4] = {gh4.x, gh4.y, gh4.z, gh4.w}, gci[4] = {gi4.x, gi4.y, gi4.z, gi4.w};
  float di[4], dO[4], du[4], df[NCH][4], dc[NCH][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float gh = (root ? 0.f : ghp[e]) + lg[e];
    const float tau = tanh_(cc[e]);
    dO[e] = gh * tau * og[e] * (1.f - og[e]);
    const float gc = (root ? 0.f : gci[e]) + gh * og[e] * (1.f - tau * tau);
    di[e] = gc * ug[e] * ig[e] * (1.f - ig[e]);
    du[e] = gc * ig[e] * (1.f - ug[e] * ug[e]);
    if constexpr (!LEAF) {
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const float fk[4] = {fk4[k].x, fk4[k].y, fk4[k].z, fk4[k].w};
        const float ck[4] = {ck4[k].x, ck4[k].y, ck4[k].z, ck4[k].w};
        df[k][e] = cp[k] >= 0 ? gc * ck[e] * fk[e] * (1.f - fk[e]) : 0.f;
        dc[k][e] = gc * fk[e];
      }
    }
  }
  auto f4 = [](const float (&x)[4]) { return make_float4(x[0], x[1], x[2], x[3]); };
  float* da = n.dA + (size_t)p * n.GW + j0;
  unsigned short* db = wb ? n.dAb + (size_t)p * n.GW + j0 : nullptr;
  auto st = [&](int col, const float (&x)[4]) {
    st4(da + col, f4(x));
    if (db) {
      *reinterpret_cast<uint2*>(db + col) = make_uint2(f2bf2(x[0], x[1]), f2bf2(x[2], x[3]));
    }
  };
  st(0, di);
  st(2 * H, dO);
  st(3 * H, du);
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const bool has = !LEAF && cp[k] >= 0;
    if (has || p >= n.f_unread_below) {
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      if constexpr (!LEAF) {
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = df[k][e];
      }
      st(f_col(k, H), z);
    }
    if constexpr (!LEAF)
      if (has) st4(n.dCp + (size_t)cp[k] * H + j0, f4(dc[k]));
  }
}

// The start of a backward, two things that only need the forward: workgroups
// below `roots` take the positions >= n.fuse_from, one each (all but the roots
// exit at once; every other position there gets its dA in the epilogue of its
// parent's level product); the rest form the h~ rows (sum of the present
// children's h) of the positions [off, off + M), dU's operand, four units a
// thread.  As two launches 5.7 + 6.6 us on the SST batch, 4.9 + 4.2 on a small
// one; so 7.2 and 4.1.
template <int NCH>
__global__ void __launch_bounds__(256) k_lstm_bwd_start(Net n, int roots, int off, int M) {
  const int H = n.H;
  if ((int)blockIdx.x < roots) {
    const int p = n.fuse_from + blockIdx.x;
    if (n.parent_pos[p] >= 0) return;
    for (int j = threadIdx.x; j < H; j += 256) lstm_gates_elem<NCH, true>(n, p, j, 0.f, 0.f);
    return;
  }
  const int q = H / 4;
  const long long i = (long long)(blockIdx.x - roots) * 256 + threadIdx.x;
  if (i >= (long long)M * q) return;
  const int p = off + (int)(i / q), j0 = 4 * (int)(i % q);
  float4 s = f4zero();
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int c = n.child_pos[(size_t)p * NCH + k];
    if (c >= 0) s = add4(s, ldg4(n.Hs + (size_t)c * H + j0));
  }
  st4(n.Ht + (size_t)p * H + j0, s);
}

// --------------------------------------------------- split-K level kernels
// For levels too small to fill the chip with the tiles above: a workgroup
// owns 16 positions x 16 units (forward) or 16 positions x 16 columns
// (backward); wavefront w accumulates the w-th quarter of the contraction.
// MFMA fragments are loaded straight from global memory into registers: in
// the permuted-K order lane group g needs k = 8g .. 8g+7 of its A row (two
// float4) and of its B column.  The four partial sums are reduced in LDS in
// a fixed order (deterministic) and the epilogue is shared with the tiled
// kernels.  BF selects bf16 operands (one 16x16x32 MFMA per 32-deep chunk)
// instead of fp32 (eight 16x16x4 steps).
template <int NCH, int TR, int KW = 4>
struct FwdRed {
  float v[KW][TR][3 + NCH][4][64];
};

// One 16*TR-position x 16-unit forward tile (row tile rt, unit tile ut).
// Wavefronts 0 .. KW-1 split the contraction.  With EPI, four more
// wavefronts (KW .. KW+3) own the epilogue: they read everything it needs
// besides the product (bias, pulled term, children's c) while the others
// multiply, then finish element i = w - KW of every row tile.  Without EPI
// (persistent loop, 64*KW threads) the contraction wavefronts finish it.
// EXACT: every share is an even number of chunks.  UT: fp32 weights from rows
// of U^T (n.UT), 16 bytes at a time, instead of down the columns of U.
template <int NCH, bool BF, int TR, int KW, bool EPI, bool EXACT = true, bool UT = false>
__device__ __forceinline__ void lstm_fwd_sk_tile(const Net& n, const RangeRows& rows, int ut,
                                                 FwdRed<NCH, TR, KW>& R) {
  constexpr int NACC = 3 + NCH;
  auto& red = R.v;
  const int H = n.H, H4 = 4 * H;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int u0 = ut * 16;
  v4f acc[TR][NACC];
  if (w < KW) {
    // A rows of this lane: the children of the position of tile row 16 tr + r.
    // An absent child (or a row past the level) reads the zero row, so the
    // loads are unconditional.
    const float* ap[TR][NCH];
#pragma unroll
    for (int tr = 0; tr < TR; ++tr) {
      const int pa = rows.pos(16 * tr + r);
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int cp = pa >= 0 ? n.child_pos[(size_t)pa * NCH + c] : -1;
        ap[tr][c] = cp >= 0 ? n.Hs + (size_t)cp * H : n.zrow;
      }
    }
    const float* ut4 = n.UT + (size_t)(u0 + r) * H;   // row u0 + r of U^T's gate block 0
    const float* ub = n.U + u0 + r;                   // column u0 + r of U's
    // this wavefront's contiguous share of the 32-deep chunks (the last
    // shares may be short or empty)
    const int nch = H / kBK, cpw = cdiv_dev(nch, KW);
    const int cbeg = min(nch, w * cpw), cend = min(nch, cbeg + cpw);
#pragma unroll
    for (int tr = 0; tr < TR; ++tr)
#pragma unroll
      for (int g = 0; g < NACC; ++g) acc[tr][g] = v4f{0.f, 0.f, 0.f, 0.f};

    // bf16: the weight fragment comes pre-rounded from n.UTb (U^T, one 16-byte
    // load per gate)
    struct Frag {
      float a[TR][NCH][8];
      float b[BF ? 1 : 4][8];
      bf16x8 bq[BF ? 4 : 1];
    };
    const u16* utb = BF ? n.UTb + (size_t)(u0 + r) * H : nullptr;
    auto load_a = [&](int k0, Frag& f) {
      const int kk = k0 + 8 * gq;
#pragma unroll
      for (int tr = 0; tr < TR; ++tr)
#pragma unroll
        for (int c = 0; c < NCH; ++c) ld8(ap[tr][c] + kk, f.a[tr][c]);
    };
    auto load_b = [&](int k0, Frag& f) {
      const int kk = k0 + 8 * gq;
      if constexpr (BF) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          f.bq[g] = *reinterpret_cast<const bf16x8*>(utb + (size_t)g * H * H + kk);
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if constexpr (UT) {
            ld8(ut4 + (size_t)g * H * H + kk, f.b[g]);
          } else {
#pragma unroll
            for (int s = 0; s < 8; ++s) f.b[g][s] = ub[(size_t)(kk + s) * H4 + g * H];
          }
        }
      }
    };
    auto load = [&](int k0, Frag& f) {
      load_a(k0, f);
      load_b(k0, f);
    };
    auto compute = [&](const Frag& f) {
#pragma unroll
      for (int tr = 0; tr < TR; ++tr) {
        const auto& a = f.a[tr];
        float ah[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          ah[s] = a[0][s];
#pragma unroll
          for (int c = 1; c < NCH; ++c) ah[s] += a[c][s];
        }
        if constexpr (BF) {
          const bf16x8 hb = to_bf8(ah);
          acc[tr][0] = mfma_bf16_16x16x32(hb, f.bq[G_I], acc[tr][0]);
          acc[tr][1] = mfma_bf16_16x16x32(hb, f.bq[G_O], acc[tr][1]);
          acc[tr][2] = mfma_bf16_16x16x32(hb, f.bq[G_U], acc[tr][2]);
#pragma unroll
          for (int c = 0; c < NCH; ++c)
            acc[tr][3 + c] = mfma_bf16_16x16x32(to_bf8(a[c]), f.bq[G_F], acc[tr][3 + c]);
        } else {
          acc[tr][0] = mfma_chunk8<BF>(ah, f.b[G_I], acc[tr][0]);
          acc[tr][1] = mfma_chunk8<BF>(ah, f.b[G_O], acc[tr][1]);
          acc[tr][2] = mfma_chunk8<BF>(ah, f.b[G_U], acc[tr][2]);
#pragma unroll
          for (int c = 0; c < NCH; ++c)
            acc[tr][3 + c] = mfma_chunk8<BF>(a[c], f.b[G_F], acc[tr][3 + c]);
        }
      }
    };
    // two register buffers: loads of the next chunk overlap the current MFMAs
    Frag fa, fb;
    if (EXACT || cbeg < cend) load(cbeg * kBK, fa);
    for (int c = cbeg; c < cend; c += 2) {
      if (EXACT || c + 1 < cend) load((c + 1) * kBK, fb);
      __builtin_amdgcn_sched_barrier(0);   // the next chunk's loads go out before these MFMAs
      compute(fa);
      if (c + 2 < cend) load((c + 2) * kBK, fa);
      if (EXACT || c + 1 < cend) compute(fb);
    }
#pragma unroll
    for (int tr = 0; tr < TR; ++tr)
#pragma unroll
      for (int g = 0; g < NACC; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          red[w][tr][g][i][lane] = acc[tr][g][i];
  }
  auto zsum = [&](int tr, int i, float (&z)[NACC]) {
#pragma unroll
    for (int g = 0; g < NACC; ++g) {
      float t = red[0][tr][g][i][lane];
#pragma unroll
      for (int q = 1; q < KW; ++q) t += red[q][tr][g][i][lane];
      z[g] = t;
    }
  };
  if constexpr (EPI) {
    const int i = w - KW;
    FwdPre<NCH> pre[TR];
    if (w >= KW) {
#pragma unroll
      for (int tr = 0; tr < TR; ++tr) {
        // rows past the level read its last row (unused), so the loads
        // are unconditional
        lstm_fwd_pre<NCH>(n, rows.clamp(16 * tr + 4 * gq + i), u0 + r, pre[tr]);
      }
    }
    __syncthreads();
    if (w < KW) return;
#pragma unroll
    for (int tr = 0; tr < TR; ++tr) {
      const int p = rows.pos(16 * tr + 4 * gq + i);
      if (p < 0) continue;
      float z[NACC], zf[NCH];
      zsum(tr, i, z);
#pragma unroll
      for (int c = 0; c < NCH; ++c) zf[c] = z[3 + c];
      lstm_fwd_fin<NCH>(n, p, u0 + r, pre[tr], z[0], z[1], z[2], zf);
    }
  } else {
    __syncthreads();
    // wave w finishes element i = w % 4 of row tiles tr = w / 4, w / 4 + KW / 4, ...
    const int i = w & 3;
#pragma unroll
    for (int tr = w >> 2; tr < TR; tr += KW / 4) {
      const int p = rows.pos(16 * tr + 4 * gq + i);
      if (p < 0) continue;
      float z[NACC], zf[NCH];
      zsum(tr, i, z);
#pragma unroll
      for (int c = 0; c < NCH; ++c) zf[c] = z[3 + c];
      lstm_fwd_epilogue<NCH>(n, p, u0 + r, z[0], z[1], z[2], zf);
    }
  }
}

template <int NCH, bool BF, int TR, int KW, bool EXACT, bool UT = false>
__global__ void __launch_bounds__(64 * (KW + 4)) k_lstm_fwd_level_sk(Net n, int off, int M) {
  __shared__ FwdRed<NCH, TR, KW> red;
  int rt, ut;
  xcd_tile(n.H / 16, rt, ut);
  lstm_fwd_sk_tile<NCH, BF, TR, KW, true, EXACT, UT>(
      n, RangeRows{off + rt * 16 * TR, off + M}, ut, red);
}

template <int NCH, int TR, int KW = 4>
struct BwdRed {
  float v[KW][TR][NCH >= 2 ? 1 + NCH : 1][4][64];
};

// One 16*TR-position x 16-column backward tile (row tile rt, column tile ut);
// wavefront roles as in the forward tile (EPI: four epilogue wavefronts
// that prefetch the children's saved state while the others multiply).
// EXACT: every wavefront's share of the contraction is a whole number of the
// groups below (H % 512 == 0 at KW = 8, H % 256 == 0 at KW = 4); otherwise
// the last shares are short: chunks past a share are loaded from a valid
// place (so that the loads of a group stay unconditional) but not multiplied.
template <int NCH, bool BF, int TR, int KW, bool EPI, bool EXACT = true>
__device__ __forceinline__ void lstm_bwd_sk_tile(const Net& n, const RangeRows& rows, int ut,
                                                 BwdRed<NCH, TR, KW>& R) {
  constexpr int NACC = NCH >= 2 ? 1 + NCH : 1;
  auto& red = R.v;
  const int H = n.H, H4 = 4 * H, GW = n.GW;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int n0 = ut * 16;
  if (w < KW) {
    // rows past the level read its last row: their sums are never used
    const float* da[TR];
    size_t daoff[TR];
#pragma unroll
    for (int tr = 0; tr < TR; ++tr) {
      daoff[tr] = (size_t)rows.clamp(16 * tr + r) * GW;
      da[tr] = n.dA + daoff[tr];
    }
    // bf16: dA's bf16 copy (written with dA, rounded as the product rounds
    // it): eight values in one 16-byte load, no conversion
    auto lda = [&](int tr, int col, float (&v)[BF ? 1 : 8], bf16x8& q) {
      if constexpr (BF) q = *reinterpret_cast<const bf16x8*>(n.dAb + daoff[tr] + col);
      else ld8(da[tr] + col, v);
    };
    // the U fragment: row n0 + r of U at columns col .. col+7
    auto ldu = [&](int col, float (&v)[8], bf16x8& q) {
      if constexpr (BF) {
        q = *reinterpret_cast<const bf16x8*>(n.Ub + (size_t)(n0 + r) * H4 + col);
      } else {
        ld8(n.U + (size_t)(n0 + r) * H4 + col, v);
      }
    };
    v4f acc[TR][NACC];
#pragma unroll
    for (int tr = 0; tr < TR; ++tr)
#pragma unroll
      for (int g = 0; g < NACC; ++g) acc[tr][g] = v4f{0.f, 0.f, 0.f, 0.f};
    // phase 1: i|o|u columns (all four blocks with one child slot)
    struct F1 {
      float a[TR][BF ? 1 : 8], b[BF ? 1 : 8];
      bf16x8 aq[TR], bq;
    };
    const int K1 = NCH == 1 ? H4 : 3 * H, q1 = cdiv_dev(K1 / kBK, KW) * kBK;
    const int beg1 = min(K1, w * q1), end1 = min(K1, beg1 + q1);
    auto load1 = [&](int c0, F1& f) {
      if (!EXACT) c0 = min(c0, K1 - kBK);
      const int col = (NCH >= 2 && c0 >= H ? c0 + H : c0) + 8 * gq;
#pragma unroll
      for (int tr = 0; tr < TR; ++tr) lda(tr, col, f.a[tr], f.aq[tr]);
      float dummy[8];
      if constexpr (BF) ldu(col, dummy, f.bq);
      else ldu(col, f.b, f.bq);
    };
    auto comp1 = [&](int c0, const F1& f) {
      if (!EXACT && c0 >= end1) return;
#pragma unroll
      for (int tr = 0; tr < TR; ++tr) {
        if constexpr (BF) acc[tr][0] = mfma_bf16_16x16x32(f.aq[tr], f.bq, acc[tr][0]);
        else acc[tr][0] = mfma_chunk8<BF>(f.a[tr], f.b, acc[tr][0]);
      }
    };
    // groups of G chunks: all loads of a group are in flight together, so a
    // small level pays about one memory latency per group, not per chunk
    constexpr int G1 = NCH >= 2 ? 6 : 8;
    if constexpr (NCH >= 2) {
      // the two phases' loads go out together: one memory latency per level
      struct F2 {
        float a[NCH][TR][BF ? 1 : 8], b[BF ? 1 : 8];
        bf16x8 aq[NCH][TR], bq;
      };
      const int q2 = cdiv_dev(H / kBK, KW) * kBK;
      const int beg2 = min(H, w * q2), end2 = min(H, beg2 + q2);
      auto load2 = [&](int c0, F2& f) {
        if (!EXACT) c0 = min(c0, H - kBK);
        const int col = c0 + 8 * gq;
#pragma unroll
        for (int tr = 0; tr < TR; ++tr)
#pragma unroll
          for (int k = 0; k < NCH; ++k) lda(tr, f_col(k, H) + col, f.a[k][tr], f.aq[k][tr]);
        float dummy[8];
        if constexpr (BF) ldu(H + col, dummy, f.bq);
        else ldu(H + col, f.b, f.bq);
      };
      auto comp2 = [&](int c0, const F2& f) {
        if (!EXACT && c0 >= end2) return;
#pragma unroll
        for (int tr = 0; tr < TR; ++tr)
#pragma unroll
          for (int k = 0; k < NCH; ++k) {
            if constexpr (BF)
              acc[tr][1 + k] = mfma_bf16_16x16x32(f.aq[k][tr], f.bq, acc[tr][1 + k]);
            else
              acc[tr][1 + k] = mfma_chunk8<BF>(f.a[k][tr], f.b, acc[tr][1 + k]);
          }
      };
      constexpr int G2 = 2;   // EXACT: H / (32 KW) is even
      // per group: the phase-2 chunks and the first half of the phase-1
      // chunks load together; the second half loads into the registers the
      // phase-2 fragments free, while the first half is multiplied
      constexpr int GH = G1 / 2;
      int c1 = beg1;
      for (int c0 = beg2; c0 < end2 || (!EXACT && c1 < end1); c0 += G2 * kBK, c1 += G1 * kBK) {
        F2 f2[G2];
        F1 fa[GH], fb[GH];
#pragma unroll
        for (int g = 0; g < G2; ++g) load2(c0 + g * kBK, f2[g]);
#pragma unroll
        for (int g = 0; g < GH; ++g) load1(c1 + g * kBK, fa[g]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < G2; ++g) comp2(c0 + g * kBK, f2[g]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < GH; ++g) load1(c1 + (GH + g) * kBK, fb[g]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < GH; ++g) comp1(c1 + g * kBK, fa[g]);
#pragma unroll
        for (int g = 0; g < GH; ++g) comp1(c1 + (GH + g) * kBK, fb[g]);
      }
    } else {
      for (int c0 = beg1; c0 < end1; c0 += G1 * kBK) {
        F1 f[G1];
#pragma unroll
        for (int g = 0; g < G1; ++g) load1(c0 + g * kBK, f[g]);
        __builtin_amdgcn_sched_barrier(0);   // keep every load of the group ahead of the MFMAs
#pragma unroll
        for (int g = 0; g < G1; ++g) comp1(c0 + g * kBK, f[g]);
      }
    }
#pragma unroll
    for (int tr = 0; tr < TR; ++tr)
#pragma unroll
      for (int g = 0; g < NACC; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[w][tr][g][i][lane] = acc[tr][g][i];
  }
  auto zsum = [&](int tr, int i, float (&z)[NACC]) {
#pragma unroll
    for (int g = 0; g < NACC; ++g) {
      float t = red[0][tr][g][i][lane];
#pragma unroll
      for (int q = 1; q < KW; ++q) t += red[q][tr][g][i][lane];
      z[g] = t;
    }
  };
  if constexpr (EPI) {
    const int i = w - KW;
    BwdPre<NCH> pre[TR];
    if (w >= KW) {
#pragma unroll
      for (int tr = 0; tr < TR; ++tr) {
        // rows past the level read its last row (unused), so the loads
        // are unconditional
        lstm_bwd_pre<NCH>(n, rows.clamp(16 * tr + 4 * gq + i), n0 + r, pre[tr]);
      }
    }
    __syncthreads();
    if (w < KW) return;
#pragma unroll
    for (int tr = 0; tr < TR; ++tr) {
      const int p = rows.pos(16 * tr + 4 * gq + i);
      if (p < 0) continue;
      float z[NACC], zf[NCH];
      zsum(tr, i, z);
#pragma unroll
      for (int k = 0; k < NCH; ++k) zf[k] = NCH >= 2 ? z[1 + k] : 0.f;
      lstm_bwd_fin<NCH>(n, p, n0 + r, pre[tr], z[0], zf);
    }
  } else {
    __syncthreads();
    const int i = w & 3;
#pragma unroll
    for (int tr = w >> 2; tr < TR; tr += KW / 4) {
      const int p = rows.pos(16 * tr + 4 * gq + i);
      if (p < 0) continue;
      float z[NACC], zf[NCH];
      zsum(tr, i, z);
#pragma unroll
      for (int k = 0; k < NCH; ++k) zf[k] = NCH >= 2 ? z[1 + k] : 0.f;
      lstm_bwd_scatter<NCH>(n, p, n0 + r, z[0], zf);
    }
  }
}

template <int NCH, bool BF, int TR, int KW, bool EXACT>
__global__ void __launch_bounds__(64 * (KW + 4)) k_lstm_bwd_level_sk(Net n, int off, int M) {
  __shared__ BwdRed<NCH, TR, KW> red;
  int rt, ut;
  xcd_tile(n.H / 16, rt, ut);
  lstm_bwd_sk_tile<NCH, BF, TR, KW, true, EXACT>(
      n, RangeRows{off + rt * 16 * TR, off + M}, ut, red);
}

// ----------------------------------------------- persistent small-level loop
// Levels shrink towards the roots (each vertex of level t+1 has its own child
// on level t), so the small levels form a suffix of the schedule.  One
// cooperative launch runs that whole suffix: tiles of a level are spread over
// the grid, and a grid barrier separates dependent levels, instead of one or
// two kernel launches per level.  Level offsets are read on the device.
//
// Grid barrier: counters only grow (zeroed before the launch).  Barrier e
// completes when the root counter reaches (e+1) * groups; the last arrival
// publishes gen = e+1.  Waiting is bounded: after `spin` polls (kBarrierSpin
// unless the CAVS_PERSIST_SPIN test hook sets another; a negative value gives
// up at once) the barrier records an error flag -- in the workspace and in
// the context's mapped host word, which cavs_sync reports -- and returns
// rather than hang.  The launch's results are then invalid.
constexpr int kBarrierSpin = 1 << 24;

struct GridBar {
  int* cnt;   // [1 + groups]: root, then one counter per group of 16 workgroups
  int* gen;
  int* err;
  int* host_err;   // mapped pinned word of the context (may be null)
  int spin;
};

__device__ __forceinline__ void grid_bar_gave_up(const GridBar& b) {
  atomicOr(b.err, 1);
  if (b.host_err) __hip_atomic_store(b.host_err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void grid_sync(const GridBar& b, int& epoch) {
  __syncthreads();
  if (threadIdx.x == 0) {
    const int G = gridDim.x, grp = blockIdx.x >> 4;
    const int gsize = min(16, G - (grp << 4)), ngroups = (G + 15) >> 4;
    __threadfence();   // release this workgroup's writes
    const int old = atomicAdd(&b.cnt[1 + grp], 1);
    bool release = false;
    if (old == epoch * gsize + gsize - 1) {
      const int o2 = atomicAdd(&b.cnt[0], 1);
      release = o2 == epoch * ngroups + ngroups - 1;
    }
    if (release) {
      __threadfence();
      atomicAdd(b.gen, 1);
    } else if (b.spin < 0) {
      grid_bar_gave_up(b);
    } else {
      int it = 0;
      while (__hip_atomic_load(b.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= epoch) {
        if (++it > b.spin) {
          grid_bar_gave_up(b);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __threadfence();   // acquire
  }
  ++epoch;
  __syncthreads();
}

template <int NCH, bool BF>
__global__ void __launch_bounds__(256) k_lstm_fwd_persist(Net n, const int* lo, int t0, int t1,
                                                          GridBar bar) {
  __shared__ FwdRed<NCH, 1> red;
  const int ut = n.H / 16;
  int epoch = 0;
  for (int t = t0; t < t1; ++t) {
    const int off = lo[t], M = lo[t + 1] - off;
    const int tiles = cdiv_dev(M, 16) * ut;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
      lstm_fwd_sk_tile<NCH, BF, 1, 4, false>(n, RangeRows{off + tile / ut * 16, off + M}, tile % ut,
                                             red);
      __syncthreads();
    }
    if (t + 1 < t1) grid_sync(bar, epoch);
  }
}

// Levels t1-1 down to t0 (all with children): the dh_k products, whose
// epilogue forms the children's dA, then a barrier.
template <int NCH, bool BF>
__global__ void __launch_bounds__(256) k_lstm_bwd_persist(Net n, const int* lo, int t0, int t1,
                                                          GridBar bar) {
  __shared__ BwdRed<NCH, 1> red;
  const int ut = n.H / 16;
  int epoch = 0;
  for (int t = t1 - 1; t >= t0; --t) {
    const int off = lo[t], M = lo[t + 1] - off;
    const int tiles = cdiv_dev(M, 16) * ut;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
      lstm_bwd_sk_tile<NCH, BF, 1, 4, false>(n, RangeRows{off + tile / ut * 16, off + M}, tile % ut,
                                             red);
      __syncthreads();
    }
    if (t > t0) grid_sync(bar, epoch);
  }
}
}  // namespace

void lstm_fwd_leaf(const Net& n, int off, int M, hipStream_t s) {
  if (M <= 0) return;
  CAVS_LAUNCH_ROWS("k_lstm_leaf", off, M, k_lstm_leaf, dim3(cdiv((long)M * n.H, 256)), dim3(256), 0,
                   s, n, off, M);
}

// bf16 levels from this many positions (below the tile threshold) run the
// split-K products with two 16-position row tiles per workgroup and four
// contraction wavefronts: each weight fragment loaded serves 32 positions,
// where the levels of 64-256 positions are bound by the operand stream.
// Measured on the H = 1024 batch: 7.60 -> 7.18 ms per step; from 32 or 96
// positions it gains less, and the smallest levels need the eight-wavefront
// split's parallelism (kSkTwoRowsFrom, kernels.h).

// Contraction wavefronts of a split-K level product: eight where each then
// has two 32-deep chunks (H % 512 == 0), or where four would have three or
// more (from H = 320); four at H = 256, whose shares are whole groups, and
// below.
// Their fp32 weights come down the columns of U, from H = 1024 (where shares
// are whole) along the rows of U^T.  us a level, columns / rows: H = 256, two
// children 5.2 / 6.2, H = 320 6.8 / 7.4, H = 768 9.3 / 10.1 (one child 8.1 /
// 9.4), H = 512 7.7 / 8.1; H = 1024 14.1 / 13.5, three children 19.8 / 17.7.
bool sk_eight(int H) { return H > 256 && (H % 256 != 0 || H % 512 == 0); }

void lstm_fwd_level(const Net& n, int off, int M, hipStream_t s) {
  if (M <= 0) return;
  if (lstm_fwd_tile_applies(n, M)) {
    lstm_fwd_tile(n, off, M, s);
    return;
  }
  const dim3 g(cdiv(M, 16) * (n.H / 16));
  const bool two = n.bf && M >= kSkTwoRowsFrom;
  // four child slots: eight contraction wavefronts would spill (168 registers each)
  const bool kw8 = !two && n.N < 4 && sk_eight(n.H);
  const bool exact = n.H % (kw8 ? 512 : 256) == 0;
#define CAVS_FWD_SK(NCH, BF, TR, KW, GRID)                                                     \
  do {                                                                                         \
    if (exact && !BF && n.H >= 1024)                                                           \
      CAVS_LAUNCH_ROWS("k_lstm_fwd_level_sk<" #NCH ", " #BF ", " #TR ", " #KW ", ut>", off, M, \
                       (k_lstm_fwd_level_sk<NCH, BF, TR, KW, true, !BF>), GRID,                 \
                       dim3(64 * (KW + 4)), 0, s, n, off, M);                                  \
    else if (exact) CAVS_LAUNCH_ROWS("k_lstm_fwd_level_sk<" #NCH ", " #BF ", " #TR ", " #KW ">", off, \
                                M, (k_lstm_fwd_level_sk<NCH, BF, TR, KW, true>), GRID,           \
                                dim3(64 * (KW + 4)), 0, s, n, off, M);                          \
    else CAVS_LAUNCH_ROWS("k_lstm_fwd_level_sk<" #NCH ", " #BF ", " #TR ", " #KW ", any>", off, \
                          M, (k_lstm_fwd_level_sk<NCH, BF, TR, KW, false>), GRID,               \
                          dim3(64 * (KW + 4)), 0, s, n, off, M);                                \
  } while (0)
#define CAVS_FWD_SK1(NCH, BF)                \
  do {                                       \
    if (kw8) CAVS_FWD_SK(NCH, BF, 1, 8, g);  \
    else CAVS_FWD_SK(NCH, BF, 1, 4, g);      \
  } while (0)
  if (two) {
    const dim3 g2(cdiv(M, 32) * (n.H / 16));
    if (n.N == 2) CAVS_FWD_SK(2, true, 2, 4, g2);
    else CAVS_FWD_SK(1, true, 2, 4, g2);
  } else if (n.N == 4) {
    CAVS_FWD_SK(4, false, 1, 4, g);
  } else if (n.N == 3) {
    CAVS_FWD_SK1(3, false);
  } else if (n.N == 2) {
    if (n.bf) CAVS_FWD_SK1(2, true);
    else CAVS_FWD_SK1(2, false);
  } else {
    if (n.bf) CAVS_FWD_SK1(1, true);
    else CAVS_FWD_SK1(1, false);
  }
#undef CAVS_FWD_SK1
#undef CAVS_FWD_SK
}

void lstm_bwd_gates(const Net& n, int off, int M, hipStream_t s) {
  if (M <= 0) return;
  // level 0 (off == 0) holds the leaves, which have no children; an internal
  // bf16 level also gets the bf16 copy of its dA (its product's operand)
  const dim3 g4(cdiv((long)M * (n.H / 4), 256));
  const int wb = n.dAb && off > 0;
#define CAVS_G4(NCH, LEAF)                                                                   \
  CAVS_LAUNCH_ROWS("k_lstm_bwd_gates4<" #NCH ", " #LEAF ">", off, M,                          \
                   (k_lstm_bwd_gates4<NCH, LEAF>), g4, dim3(256), 0, s, n, off, M, wb)
  if (n.N == 4) {
    if (off == 0) CAVS_G4(4, true);
    else CAVS_G4(4, false);
  } else if (n.N == 3) {
    if (off == 0) CAVS_G4(3, true);
    else CAVS_G4(3, false);
  } else if (n.N == 2) {
    if (off == 0) CAVS_G4(2, true);
    else CAVS_G4(2, false);
  } else {
    if (off == 0) CAVS_G4(1, true);
    else CAVS_G4(1, false);
  }
#undef CAVS_G4
}

void lstm_bwd_start(const Net& n, int off, hipStream_t s) {
  const int roots = n.V - n.fuse_from, M = n.Ht ? n.V - off : 0;
  const dim3 g(roots + cdiv((long)M * (n.H / 4), 256));
  if (g.x == 0) return;
#define CAVS_START(NCH) \
  CAVS_LAUNCH("k_lstm_bwd_start", k_lstm_bwd_start<NCH>, g, dim3(256), 0, s, n, roots, off, M)
  if (n.N == 4) CAVS_START(4);
  else if (n.N == 3) CAVS_START(3);
  else if (n.N == 2) CAVS_START(2);
  else CAVS_START(1);
#undef CAVS_START
}

int lstm_fuse_level(const int* lo_host, int T) {
  for (int t = 0; t < T; ++t)
    if (lo_host[t + 1] - lo_host[t] <= kFuseRows) return t;
  return T;
}

void lstm_bwd_level(const Net& n, int off, int M, hipStream_t s) {
  if (M <= 0) return;
  if (lstm_bwd_tile_applies(n, M)) {
    lstm_bwd_tile(n, off, M, s);
    return;
  }
  const dim3 g(cdiv(M, 16) * (n.H / 16));
  const bool two = n.bf && M >= kSkTwoRowsFrom;
  // eight K wavefronts at most 128 positions (one round); four above, where
  // two workgroups per CU keep the whole level co-resident
  const bool kw8 = !two && sk_eight(n.H) && M <= 128;
  const bool exact = n.H % (kw8 ? 512 : 256) == 0;
#define CAVS_BWD_SK(NCH, BF, TR, KW, GRID)                                                     \
  do {                                                                                         \
    if (exact) CAVS_LAUNCH_ROWS("k_lstm_bwd_level_sk<" #NCH ", " #BF ", " #TR ", " #KW ">", off, \
                                M, (k_lstm_bwd_level_sk<NCH, BF, TR, KW, true>), GRID,           \
                                dim3(64 * (KW + 4)), 0, s, n, off, M);                          \
    else CAVS_LAUNCH_ROWS("k_lstm_bwd_level_sk<" #NCH ", " #BF ", " #TR ", " #KW ", any>", off, \
                          M, (k_lstm_bwd_level_sk<NCH, BF, TR, KW, false>), GRID,               \
                          dim3(64 * (KW + 4)), 0, s, n, off, M);                                \
  } while (0)
#define CAVS_BWD_SK1(NCH, BF)                \
  do {                                       \
    if (kw8) CAVS_BWD_SK(NCH, BF, 1, 8, g);  \
    else CAVS_BWD_SK(NCH, BF, 1, 4, g);      \
  } while (0)
  if (two) {
    const dim3 g2(cdiv(M, 32) * (n.H / 16));
    if (n.N == 2) CAVS_BWD_SK(2, true, 2, 4, g2);
    else CAVS_BWD_SK(1, true, 2, 4, g2);
  } else if (n.N == 4) {
    CAVS_BWD_SK1(4, false);
  } else if (n.N == 3) {
    CAVS_BWD_SK1(3, false);
  } else if (n.N == 2) {
    if (n.bf) CAVS_BWD_SK1(2, true);
    else CAVS_BWD_SK1(2, false);
  } else {
    if (n.bf) CAVS_BWD_SK1(1, true);
    else CAVS_BWD_SK1(1, false);
  }
#undef CAVS_BWD_SK1
#undef CAVS_BWD_SK
}

namespace {

// Levels of at most this many positions run in the persistent loop.
constexpr int kPersistRows = 256;

// The persistent loop is an opt-in ablation (CAVS_PERSIST=1): measured on
// MI355X, one grid barrier with the agent-scope fences it needs costs
// 2.7-17 us (32-512 workgroups) against 2.4 us for a back-to-back kernel
// launch, so per-level launches are the default.
bool persist_enabled() {
  const char* e = getenv("CAVS_PERSIST");
  return e && e[0] && e[0] != '0';
}

int coresident_blocks(const void* fn) {
  static std::map<const void*, int> cache;
  auto it = cache.find(fn);
  if (it != cache.end()) return it->second;
  int dev = 0, ncu = 0, per = 0, coop = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, 256, 0) != hipSuccess || !coop)
    per = 0;
  const int v = per * ncu;
  cache[fn] = v;
  return v;
}

bool launch_persist(const char* name, const void* fn, const Net& n, const int* lo,
                    const int* lo_host, int t0, int t1, int* bar, int max_rows, hipStream_t s) {
  const int tiles = cdiv(max_rows, 16) * (n.H / 16);
  int G = coresident_blocks(fn);
  if (G > 512) G = 512;
  if (G > tiles) G = tiles;
  if (G <= 0) return false;
  int spin = kBarrierSpin;
  if (const char* e = getenv("CAVS_PERSIST_SPIN")) spin = atoi(e);
  GridBar gb{bar, bar + 64, bar + 65, t_active_ctx->dev_err_dev, spin};
  void* args[] = {(void*)&n, (void*)&lo, (void*)&t0, (void*)&t1, (void*)&gb};
  const LoopTurn turn(t_active_ctx->device, s);
  if (!turn.ok()) return false;
  if (zero_async(bar, 256 * sizeof(int), s) != hipSuccess) return false;
  TimedScope ts(name, s, lo_host[t0], lo_host[t1] - lo_host[t0], /*bracket=*/true);
  return hipLaunchCooperativeKernel(fn, dim3(G), dim3(256), args, 0, s) == hipSuccess;
}

}  // namespace

int persist_first_level(const Net& n, const int* lo_host, int T) {
  if (!persist_enabled() || n.H % 256 != 0 || n.N > 2) return T;
  for (int t = 1; t < T; ++t)
    if (lo_host[t + 1] - lo_host[t] <= kPersistRows) return t;
  return T;
}

bool lstm_fwd_persist(const Net& n, const int* lo, const int* lo_host, int t0, int t1, int* bar,
                      hipStream_t s) {
  if (t0 >= t1) return true;
  const int maxM = lo_host[t0 + 1] - lo_host[t0];
#define CAVS_FP(NCH, BF)                                                                   \
  launch_persist("k_lstm_fwd_persist<" #NCH ", " #BF ">",                                  \
                 reinterpret_cast<const void*>(&k_lstm_fwd_persist<NCH, BF>), n, lo, lo_host, \
                 t0, t1, bar, maxM, s)
  if (n.N == 2) return n.bf ? CAVS_FP(2, true) : CAVS_FP(2, false);
  return n.bf ? CAVS_FP(1, true) : CAVS_FP(1, false);
#undef CAVS_FP
}

bool lstm_bwd_persist(const Net& n, const int* lo, const int* lo_host, int t0, int t1, int* bar,
                      hipStream_t s) {
  if (t0 >= t1) return true;
  const int maxM = lo_host[t0 + 1] - lo_host[t0];
#define CAVS_BP(NCH, BF)                                                                   \
  launch_persist("k_lstm_bwd_persist<" #NCH ", " #BF ">",                                  \
                 reinterpret_cast<const void*>(&k_lstm_bwd_persist<NCH, BF>), n, lo, lo_host, \
                 t0, t1, bar, maxM, s)
  if (n.N == 2) return n.bf ? CAVS_BP(2, true) : CAVS_BP(2, false);
  return n.bf ? CAVS_BP(1, true) : CAVS_BP(1, false);
#undef CAVS_BP
}

}  // namespace cavs

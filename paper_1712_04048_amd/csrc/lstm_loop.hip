// XCD-local small-level loop: the small levels near the roots in one launch
// per direction, without grid-wide barriers.  The graphs of a batch are
// independent, so the top of every tree (its positions in the suffix of small
// levels) is given to one of the eight XCDs, and the workgroups running on an
// XCD (its hardware id read from XCC_ID) process only their XCD's positions,
// level by level, separated by a barrier among themselves.  Everything one
// level writes and the next reads then stays inside one XCD: its CUs share
// one L2, stores reach it through the write-through L1, and the readers'
// device-scope loads (sc1) miss their own L1 and read it.
//
// A level is a chain of latencies (children's rows, product, sum over the
// wavefronts, gates, stores, barrier), and everything that need not be on it
// is taken off:
//   - workgroup `rank` of an XCD owns 16 units (bf16 above 512: 32, in two unit
//     tiles that share the operand rows) for the whole loop and holds
//     its share of the weights in registers, split into bf16 parts
//     (split3.h): a 16-row tile's product takes 96 cycles a block instead of
//     256 on the fp32 instruction, and no weight is read again (but what
//     spills, see xcd_applies);
//   - what the next level reads that does not depend on this one (its list of
//     positions, child positions, pulled terms; backward: the children's
//     saved state) is fetched while the barrier is pending;
//   - only the stores that the next level reads precede the barrier's arrival
//     (h and c; backward: the split dA rows and dL/dc), the rest follow it;
//   - backward, a child's dA is split once, where it is formed, so that the
//     32 workgroups that read it as an operand load fragments as they are, and
//     all eight wavefronts finish children (four for each of two: with four
//     doing it all, two slots needed 19 registers more than there are and four
//     slots 62; SST batch 115 -> 98 us, trees at H = 320 253 -> 202, four slots
//     125 -> 68);
//   - the barrier is one store to the workgroup's own flag and a poll of all
//     the XCD's flags (one 128-byte line), no read-modify-write.
// Per level, 64 chains at H = 512: forward 5.4 -> 3.2 us, backward 6.2 -> 4.7
// (before: weights in LDS, fp32 instruction, counter barrier, every store
// before it).  bf16 at H = 1024 (left-branching trees, up to 16 384 positions
// over some 115 levels of 256 rows and fewer): forward 7.9, backward 9.9 us per
// level (level kernels: 10 to 30 and 12 to 29).
#include <stdlib.h>

#include "lstm_dev.h"
#include "split3.h"

namespace cavs {
namespace {

constexpr int kXcdRows = 256;          // levels of at most this many positions
constexpr int kXcdMaxSuffix = 16384;   // suffix positions the owner kernel holds
constexpr int kXcdWords = 1024;        // barrier words
constexpr int kXcdSpin = 1 << 21;      // bounded waits (polls) before giving up
constexpr int kXcdKW = 8;              // wavefronts, each a share of the contraction

// Barrier words: [0] grid arrivals, [1] grid generation, [2] error, [32 + x]
// the ticket (rank counter) of XCD x, [40 + x] its workgroups, [64 + 32 x + r]
// the barrier flag of its workgroup r: the barriers passed so far.  Arrivals
// and tickets return to zero by themselves; every flag of an XCD ends a launch
// at the same value, from which the next launch counts on.  The owner kernel zeroes them all.
struct XcdLoop {
  int* w;
  const unsigned char* own;   // owner XCD of suffix position p (indexed p - base)
  int base;
  int spin;
  int* host_err;              // mapped pinned error word of the context (may be null)
};

__device__ __forceinline__ int xcc_id() {
  int v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 7;
}

__device__ __forceinline__ int ld_sc1(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void xcd_gave_up(const XcdLoop& xl) {
  atomicOr(&xl.w[2], 1);
  if (xl.host_err) __hip_atomic_store(xl.host_err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Owner of every suffix position: the rank of its tree's root among the
// suffix roots (in position order), modulo 8.  Roots by pointer doubling in
// LDS (a parent always lies in the suffix: it is on a higher level).  One
// workgroup; also clears the barrier words.
__global__ void __launch_bounds__(1024) k_xcd_owner(const int* __restrict__ parent_pos, int base,
                                                    int S, unsigned char* __restrict__ own,
                                                    int* __restrict__ words) {
  __shared__ short ra[kXcdMaxSuffix], rb[kXcdMaxSuffix];
  __shared__ int wcnt[16], changed[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < kXcdWords; i += 1024) words[i] = 0;
  for (int q = tid; q < S; q += 1024) {
    const int pp = parent_pos[base + q];
    ra[q] = (short)(pp >= base && pp < base + S ? pp - base : q);
  }
  if (tid < 2) changed[tid] = 0;
  __syncthreads();
  short* a = ra;
  short* b = rb;
  for (int it = 0; it < 16; ++it) {   // 2^15 > kXcdMaxSuffix: enough rounds
    int ch = 0;
    for (int q = tid; q < S; q += 1024) {
      const short v = a[a[q]];
      b[q] = v;
      ch |= v != a[q];
    }
    if (ch) changed[it & 1] = 1;
    __syncthreads();
    const bool more = changed[it & 1] != 0;
    if (tid == 0) changed[(it + 1) & 1] = 0;
    short* t = a;
    a = b;
    b = t;
    __syncthreads();
    if (!more) break;
  }
  // ranks of the roots (a[q] == q) in position order: each thread a
  // contiguous chunk, a block-wide exclusive scan of the chunk counts
  const int per = (S + 1023) / 1024, q0 = min(S, tid * per), q1 = min(S, q0 + per);
  int c = 0;
  for (int q = q0; q < q1; ++q) c += a[q] == q;
  int incl = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wcnt[wv] = incl;
  __syncthreads();
  int rank = incl - c;
  for (int k = 0; k < wv; ++k) rank += wcnt[k];
  for (int q = q0; q < q1; ++q)
    if (a[q] == q) b[q] = (short)(rank++);
  __syncthreads();
  for (int q = tid; q < S; q += 1024) own[q] = (unsigned char)(b[a[q]] & 7);
}

// State of a workgroup in the loop (LDS).
struct XcdState {
  int x, rank, n, g0, epoch, err;
};

// Group formation: rank of this workgroup among those on its XCD (known at
// once), then, after a one-time grid-wide arrival, their number (every ticket
// is final).  Work that needs only the rank runs between the two halves.
__device__ __forceinline__ void xcd_arrive(const XcdLoop& xl, XcdState& s) {
  if (threadIdx.x == 0) {
    const int x = xcc_id();
    const int rank = atomicAdd(&xl.w[32 + x], 1);
    const int g0 = ld_sc1(&xl.w[1]);
    __builtin_amdgcn_s_waitcnt(0);
    const int old = atomicAdd(&xl.w[0], 1);
    if (old == (int)gridDim.x - 1) {
      // every ticket is final: keep the counts, clear the tickets
      for (int i = 0; i < 8; ++i)
        __hip_atomic_store(&xl.w[40 + i], atomicExch(&xl.w[32 + i], 0), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      atomicExch(&xl.w[0], 0);
      __builtin_amdgcn_s_waitcnt(0);
      atomicAdd(&xl.w[1], 1);
      s.g0 = -1;   // released the grid: nothing to wait for
    } else {
      s.g0 = g0;
    }
    s.x = x;
    s.rank = rank;
  }
  __syncthreads();
}

__device__ __forceinline__ void xcd_wait(const XcdLoop& xl, XcdState& s) {
  if (threadIdx.x == 0) {
    const int x = s.x, g0 = s.g0;
    if (g0 != -1) {
      int it = 0;
      while (ld_sc1(&xl.w[1]) == g0) {
        if (++it > xl.spin || ld_sc1(&xl.w[2])) {
          xcd_gave_up(xl);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    s.n = ld_sc1(&xl.w[40 + x]);
    s.epoch = s.rank < 32 ? ld_sc1(&xl.w[64 + 32 * x + s.rank]) : 0;
    s.err = ld_sc1(&xl.w[2]);
  }
  __syncthreads();
}

// Barrier among the np participating workgroups of an XCD.  Arrive: every
// store of this workgroup has reached the L2, then its flag says so.
__device__ __forceinline__ void xcd_barrier_arrive(const XcdLoop& xl, XcdState& s) {
  __builtin_amdgcn_s_waitcnt(0);   // this wavefront's stores have reached the L2
  __syncthreads();
  if (threadIdx.x == 0) {
    const int e = s.epoch + 1;
    s.epoch = e;
    __hip_atomic_store(&xl.w[64 + 32 * s.x + s.rank], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Leave: wavefront 0 polls the flags; s.err is set when the wait gave up (its
// own bound, or another workgroup's recorded error).
__device__ __forceinline__ void xcd_barrier_wait(const XcdLoop& xl, XcdState& s, int np) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x, e = s.epoch;
    const int* p = lane < np ? &xl.w[64 + 32 * s.x + lane] : &xl.w[2];
    int it = 0;
    while (true) {
      const int v = ld_sc1(p);
      const bool late = lane < np && v - e < 0, bad = lane >= np && v != 0;
      if (__ballot(late) == 0) break;
      if (++it > xl.spin || __ballot(bad) != 0) {
        if (lane == 0) {
          xcd_gave_up(xl);
          s.err = 1;
        }
        break;
      }
    }
  }
  __syncthreads();
}

// This XCD's positions of the level [l0, l1) (offsets from l0, in order)
// into lst and their number into *m; one wavefront.
__device__ __forceinline__ void xcd_level_list(const XcdLoop& xl, int x, int l0, int l1,
                                               short* lst, int* m) {
  const int lane = threadIdx.x & 63;
  int cnt = 0;
  for (int i0 = l0; i0 < l1; i0 += 64) {
    const int p = i0 + lane;
    const bool mine = p < l1 && xl.own[p - xl.base] == x;
    const unsigned long long bal = __ballot(mine);
    if (mine) lst[cnt + __popcll(bal & ((1ull << lane) - 1ull))] = (short)(p - l0);
    cnt += __popcll(bal);
  }
  if (lane == 0) *m = cnt;
}

// Parts of an operand: three in fp32 (their six products, smallest first),
// one, rounded, in bf16.
template <bool BF>
struct Parts {
  static constexpr int N = BF ? 1 : 3, TERMS = BF ? 1 : kSplitTerms;
  static constexpr int TA[6] = {BF ? 0 : 2, 0, 1, 1, 0, 0}, TB[6] = {0, 2, 1, 0, 1, 0};
};
template <bool BF>
struct Frag {
  bf16x8 p[Parts<BF>::N];
};
template <bool BF>
__device__ __forceinline__ Frag<BF> to_frag(const float (&v)[8]) {
  Frag<BF> f;
  if constexpr (BF) {
    f.p[0] = to_bf8(v);
  } else {
    const Split8 s = split8(v);
#pragma unroll
    for (int k = 0; k < 3; ++k) f.p[k] = __builtin_bit_cast(bf16x8, s.p[k]);
  }
  return f;
}

// ------------------------------------------------------------------ forward
// CPW: 32-deep chunks of the contraction per wavefront (1 up to H = 256, 2 up
// to 512, else 4); with H below 256 CPW the last wavefronts have none.  UT: unit
// tiles of the workgroup; wavefronts 4 ut .. 4 ut + 3 finish tile ut.
template <int NCH, bool BF, int CPW, int UT>
__global__ void __launch_bounds__(64 * kXcdKW, 2) k_lstm_fwd_xcd(Net n, const int* lo, int t0,
                                                                int t1, XcdLoop xl) {
  constexpr int KW = kXcdKW, NACC = 3 + NCH, EW = 4 * UT;   // EW: wavefronts of the epilogue
  using PT = Parts<BF>;
  __shared__ float red[KW][UT * NACC][4][64];
  __shared__ short lst[2][kXcdRows];
  __shared__ int sm[2];
  __shared__ XcdState s;
  xcd_arrive(xl, s);
  const int H = n.H, nut = H / (16 * UT), nch = H / kBK;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int u0 = 16 * UT * min(s.rank, nut - 1);
  const int ut = UT == 1 ? 0 : w >> 2, wr = w & 3, uj = u0 + 16 * ut + r;   // the epilogue's
  // this unit tile's weights, while the grid-wide arrival completes: columns
  // u0 + r of each gate block of U at k = 32 c + 8 gq ..
  Frag<BF> W[UT][CPW][4];
#pragma unroll
  for (int q = 0; q < UT; ++q)
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int c = min(w * CPW + i, nch - 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const size_t e = (size_t)(g * H + u0 + 16 * q + r) * H + c * kBK + 8 * gq;
        if constexpr (BF) {
          W[q][i][g].p[0] = *reinterpret_cast<const bf16x8*>(n.UTb + e);
        } else {
          float v[8];
          ld8(n.UT + e, v);
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] = split_clamp(v[x]);
          W[q][i][g] = to_frag<BF>(v);
        }
      }
    }
  const float bi = n.b[G_I * H + uj], bf = n.b[G_F * H + uj];
  const float bo = n.b[G_O * H + uj], bu = n.b[G_U * H + uj];
  xcd_wait(xl, s);
  if (s.rank >= nut) return;   // more workgroups than unit tiles: nothing to do
  if (s.n < nut) {             // fewer (the host's occupancy check excludes it): record it
    if (tid == 0) xcd_gave_up(xl);
    return;
  }
  const int x = s.x;
  const CohBuf hb = coh_buf(n.Hs, (size_t)n.V * H), cb = coh_buf(n.Cs, (size_t)n.V * H);

  // What a tile reads that no level of this launch writes: per lane the
  // child positions of tile row r, and in the epilogue's wavefronts its
  // operands of row 4 gq + wr, unit uj.
  struct Stat {
    int cr[NCH], cp[NCH], v, pulled;
    float pi, pf, po, pu;
  };
  auto fetch = [&](const ListRows& rows, Stat& q) {
    const int pa = rows.clamp(r);
#pragma unroll
    for (int k = 0; k < NCH; ++k) q.cr[k] = n.child_pos[(size_t)pa * NCH + k];
    if (w < EW) {
      const int p = rows.clamp(4 * gq + wr), j = uj;
#pragma unroll
      for (int k = 0; k < NCH; ++k) q.cp[k] = n.child_pos[(size_t)p * NCH + k];
      q.v = n.order[p];
      q.pulled = n.pull_pos[p] >= 0;
      const float* P = n.P + (size_t)p * 4 * H + j;   // an unused row where nothing is pulled
      q.pi = P[G_I * H];
      q.pf = P[G_F * H];
      q.po = P[G_O * H];
      q.pu = P[G_U * H];
    }
  };
  // results whose stores may follow the barrier's arrival
  struct Late {
    int p;
    float ig, og, ug, f[NCH], h, c;
    int v;
  } late;
  late.p = -1;
  auto flush = [&]() {
    if (late.p < 0) return;
    const int j = uj;
    if (n.Gs) {   // null in inference: nothing reads the gates back
      float* g = n.Gs + (size_t)late.p * n.GW;
      g[j] = late.ig;
      g[2 * H + j] = late.og;
      g[3 * H + j] = late.ug;
#pragma unroll
      for (int k = 0; k < NCH; ++k) g[f_col(k, H) + j] = late.f[k];
    }
    n.h_out[(size_t)late.v * H + j] = late.h;
    if (n.c_out) n.c_out[(size_t)late.v * H + j] = late.c;
    late.p = -1;
  };

  int l0 = lo[t0], l1 = lo[t0 + 1], l2 = t0 + 1 < t1 ? lo[t0 + 2] : l1;
  if (w == KW - 1) xcd_level_list(xl, x, l0, l1, lst[0], &sm[0]);
  __syncthreads();
  Stat st;
  if (sm[0] > 0) fetch(ListRows{lst[0], sm[0], l0}, st);
  for (int t = t0; t < t1 && !s.err; ++t) {
    const int cur = (t - t0) & 1, m = sm[cur];
    if (m == 0) break;   // the XCD's trees have ended (no higher level has positions either)
    const int l3 = t + 2 < t1 ? lo[t + 3] : l2;
    for (int rt = 0; 16 * rt < m; ++rt) {
      const ListRows rows{lst[cur] + 16 * rt, m - 16 * rt, l0};
      if (rt > 0) fetch(rows, st);
      constexpr int AW = CPW < 2 ? CPW : 2;   // chunks in flight
      float a[AW][NCH][8];
      auto load = [&](int i) {
        const int kk = min(w * CPW + i, nch - 1) * kBK + 8 * gq;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
          const size_t o = (size_t)max(st.cr[k], 0) * H + kk;
          const float4 y0 = coh_ld4(hb, o), y1 = coh_ld4(hb, o + 4);
          float* d = a[i % AW][k];
          d[0] = y0.x; d[1] = y0.y; d[2] = y0.z; d[3] = y0.w;
          d[4] = y1.x; d[5] = y1.y; d[6] = y1.z; d[7] = y1.w;
        }
      };
#pragma unroll
      for (int i = 0; i < AW; ++i) load(i);
      float cc[NCH];
      if (w < EW) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) cc[k] = coh_ld1(cb, (size_t)max(st.cp[k], 0) * H + uj);
      }
      v4f acc[UT][NACC];
#pragma unroll
      for (int q = 0; q < UT; ++q)
#pragma unroll
        for (int g = 0; g < NACC; ++g) acc[q][g] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        if (w * CPW + i >= nch) break;   // uniform in the wavefront
        float ah[8];
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
          const bool on = st.cr[k] >= 0;   // an absent child reads row 0: a select, that may hold NaN
          float* d = a[i % AW][k];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            d[e] = on ? d[e] : 0.f;
            ah[e] = k == 0 ? d[e] : ah[e] + d[e];
          }
        }
        const Frag<BF> fh = to_frag<BF>(ah);
        Frag<BF> fk[NCH];
        if constexpr (NCH > 1) {
#pragma unroll
          for (int k = 0; k < NCH; ++k) fk[k] = to_frag<BF>(a[i % AW][k]);
        } else {
          fk[0] = fh;
        }
        if constexpr (CPW > AW) {
          __builtin_amdgcn_sched_barrier(0);
          if (i + AW < CPW) load(i + AW);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < PT::TERMS; ++q)
#pragma unroll
          for (int e = 0; e < UT; ++e) {
            const Frag<BF>* We = W[e][i];
            acc[e][0] = mfma_bf16_16x16x32(fh.p[PT::TA[q]], We[G_I].p[PT::TB[q]], acc[e][0]);
            acc[e][1] = mfma_bf16_16x16x32(fh.p[PT::TA[q]], We[G_O].p[PT::TB[q]], acc[e][1]);
            acc[e][2] = mfma_bf16_16x16x32(fh.p[PT::TA[q]], We[G_U].p[PT::TB[q]], acc[e][2]);
#pragma unroll
            for (int k = 0; k < NCH; ++k)
              acc[e][3 + k] =
                  mfma_bf16_16x16x32(fk[k].p[PT::TA[q]], We[G_F].p[PT::TB[q]], acc[e][3 + k]);
          }
      }
#pragma unroll
      for (int q = 0; q < UT; ++q)
#pragma unroll
        for (int g = 0; g < NACC; ++g)
#pragma unroll
          for (int i = 0; i < 4; ++i) red[w][q * NACC + g][i][lane] = acc[q][g][i];
      __syncthreads();
      if (w < EW) {
        const int p = rows.pos(4 * gq + wr);
        float z[NACC];
#pragma unroll
        for (int g = 0; g < NACC; ++g) {
          z[g] = red[0][ut * NACC + g][wr][lane];
#pragma unroll
          for (int q = 1; q < KW; ++q) z[g] += red[q][ut * NACC + g][wr][lane];
        }
        if constexpr (UT == 2) flush();   // an earlier tile of this level
        if (p >= 0) {
          float ai = z[0] + bi, ao = z[1] + bo, au = z[2] + bu;
          if (st.pulled) {
            ai += st.pi;
            ao += st.po;
            au += st.pu;
          }
          const float fb = st.pulled ? bf + st.pf : bf;
          late.ig = sigmoidf_(ai);
          late.og = sigmoidf_(ao);
          late.ug = tanh_(au);
          float c = late.ig * late.ug;
#pragma unroll
          for (int k = 0; k < NCH; ++k) {
            late.f[k] = 0.f;
            if (st.cp[k] >= 0) {
              late.f[k] = sigmoidf_(z[3 + k] + fb);
              c += late.f[k] * cc[k];
            }
          }
          late.c = c;
          late.h = late.og * tanh_(c);
          late.p = p;
          late.v = st.v;
          n.Hs[(size_t)p * H + uj] = late.h;
          n.Cs[(size_t)p * H + uj] = c;
        }
      }
      if (w == KW - 1 && rt == 0 && t + 1 < t1) {
        xcd_level_list(xl, x, l1, l2, lst[cur ^ 1], &sm[cur ^ 1]);
      }
      if (16 * (rt + 1) < m) {
        if constexpr (UT == 1) flush();   // (kept over the next product it takes registers there)
        __syncthreads();                  // red is read before the next tile writes it
      }
    }
    if (t + 1 < t1) {
      xcd_barrier_arrive(xl, s);
      flush();
      l0 = l1;
      l1 = l2;
      l2 = l3;
      if (sm[cur ^ 1] > 0) fetch(ListRows{lst[cur ^ 1], sm[cur ^ 1], l0}, st);
      xcd_barrier_wait(xl, s, nut);
    }
  }
  flush();
}

// ----------------------------------------------------------------- backward
// Top level first: the workgroup owns output columns u0 .. u0 + 16 UT - 1 (rows of U
// in registers) and runs every row tile of its XCD's positions of a level;
// each child's dA (or, below the fused levels, its dL/dh) is finished in the
// epilogue.  Operand rows: n.dAp, dA's three bf16 parts (n.dAb in bf16).
template <int NCH, bool BF, int CPW, int UT>
__global__ void __launch_bounds__(64 * kXcdKW, 2) k_lstm_bwd_xcd(Net n, const int* lo, int t0,
                                                                int t1, XcdLoop xl) {
  constexpr int KW = kXcdKW, NGA = 3 + NCH, NACC = NCH >= 2 ? 1 + NCH : 1;
  // the epilogue: a wavefront finishes a quarter of a unit tile's elements; with
  // one unit tile the children are shared between two sets of four
  constexpr int KG = UT == 1 && NCH > 1 ? 2 : 1, KC = (NCH + KG - 1) / KG, EW = 4 * UT * KG;
  using PT = Parts<BF>;
  __shared__ float red[KW][UT * NACC][4][64];
  __shared__ short lst[2][kXcdRows];
  __shared__ int sm[2];
  __shared__ XcdState s;
  xcd_arrive(xl, s);
  const int H = n.H, GW = n.GW, nut = H / (16 * UT), nch = H / kBK;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, gq = lane >> 4, r = lane & 15;
  const int u0 = 16 * UT * min(s.rank, nut - 1);
  const int ut = UT == 1 ? 0 : w >> 2, wr = w & 3, uj = u0 + 16 * ut + r;   // the epilogue's
  const int kc0 = KG == 1 ? 0 : (w >> 2) * KC;                              // first child
  Frag<BF> W[UT][CPW][4];   // i, o, u, f
#pragma unroll
  for (int q = 0; q < UT; ++q)
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int c = min(w * CPW + i, nch - 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int G = g == 0 ? G_I : g == 1 ? G_O : g == 2 ? G_U : G_F;
        const size_t e = (size_t)(u0 + 16 * q + r) * 4 * H + G * H + c * kBK + 8 * gq;
        if constexpr (BF) {
          W[q][i][g].p[0] = *reinterpret_cast<const bf16x8*>(n.Ub + e);
        } else {
          float v[8];
          ld8(n.U + e, v);
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] = split_clamp(v[x]);
          W[q][i][g] = to_frag<BF>(v);
        }
      }
    }
  xcd_wait(xl, s);
  if (s.rank >= nut) return;
  if (s.n < nut) {
    if (tid == 0) xcd_gave_up(xl);
    return;
  }
  const int x = s.x, pbase = BF ? 0 : n.dAp_base;
  const size_t plane = n.dAp_plane;
  const CohBuf ab = BF ? coh_buf(reinterpret_cast<const float*>(n.dAb), (size_t)n.V * GW / 2)
                       : coh_buf(reinterpret_cast<const float*>(n.dAp), 3 * plane / 2);
  const CohBuf gb = coh_buf(n.dCp, (size_t)n.V * H);

  // children's saved state, which the forward left: the epilogue's row
  // 4 gq + wr, unit uj (an absent child, or one below the fused levels,
  // reads row 0, unused)
  struct Stat {
    int cp[KC];
    GatePre<NCH> q[KC];
  };
  auto fetch = [&](const ListRows& rows, Stat& st) {
    if (w >= EW) return;
    const int p = rows.clamp(4 * gq + wr), j = uj;
#pragma unroll
    for (int k = 0; k < KC; ++k)
      st.cp[k] = kc0 + k < NCH ? n.child_pos[(size_t)p * NCH + kc0 + k] : -1;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int c = st.cp[k] >= n.fuse_from ? st.cp[k] : 0;
      lstm_gates_pre_all<NCH, false>(n, c, j, st.q[k]);
    }
  };
  struct Late {
    int p[KC];
    float d[KC][NGA];
  } late;
#pragma unroll
  for (int k = 0; k < KC; ++k) late.p[k] = -1;
  auto flush = [&]() {
    const int j = uj;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      if (late.p[k] < 0) continue;
      float* da = n.dA + (size_t)late.p[k] * GW;
#pragma unroll
      for (int g = 0; g < NGA; ++g) da[g * H + j] = late.d[k][g];
      late.p[k] = -1;
    }
  };

  int l0 = lo[t1 - 1], l1 = lo[t1], lm = t1 - 1 > t0 ? lo[t1 - 2] : l0;
  if (w == KW - 1) xcd_level_list(xl, x, l0, l1, lst[0], &sm[0]);
  __syncthreads();
  Stat st;
  if (sm[0] > 0) fetch(ListRows{lst[0], sm[0], l0}, st);
  for (int t = t1 - 1; t >= t0 && !s.err; --t) {
    const int cur = (t1 - 1 - t) & 1, m = sm[cur];
    const int lmm = t - 2 >= t0 ? lo[t - 2] : lm;
    for (int rt = 0; 16 * rt < m; ++rt) {
      const ListRows rows{lst[cur] + 16 * rt, m - 16 * rt, l0};
      if (rt > 0) fetch(rows, st);
      const size_t row = (size_t)(rows.clamp(r) - pbase) * GW;
      // dA blocks i, o, u (a = 0, 1, 2) and f_k (3 + k) of chunk i
      auto load = [&](int i, int a, Frag<BF>& f) {
        const int col = (a == 0 ? 0 : a < 3 ? (a + 1) * H : f_col(a - 3, H)) +
                        min(w * CPW + i, nch - 1) * kBK + 8 * gq;
#pragma unroll
        for (int q = 0; q < PT::N; ++q)
          f.p[q] = __builtin_bit_cast(bf16x8, coh_ld4(ab, (q * plane + row + col) / 2));
      };
      v4f acc[UT][NACC];
#pragma unroll
      for (int q = 0; q < UT; ++q)
#pragma unroll
        for (int g = 0; g < NACC; ++g) acc[q][g] = v4f{0.f, 0.f, 0.f, 0.f};
      auto mul = [&](int i, int a0, int na, const Frag<BF>* f) {
        if (w * CPW + i >= nch) return;
#pragma unroll
        for (int q = 0; q < PT::TERMS; ++q)
#pragma unroll
          for (int a = 0; a < na; ++a) {
            const int g = a0 + a, d = NCH >= 2 && g >= 3 ? g - 2 : 0;
#pragma unroll
            for (int e = 0; e < UT; ++e)
              acc[e][d] = mfma_bf16_16x16x32(f[a].p[PT::TA[q]], W[e][i][g < 3 ? g : 3].p[PT::TB[q]],
                                             acc[e][d]);
          }
      };
      float gc[KC];
      if constexpr (CPW == 4) {   // bf16: two chunks' rows in flight
        Frag<BF> f[2][NGA];
        auto load_all = [&](int i) {
#pragma unroll
          for (int a = 0; a < NGA; ++a) load(i, a, f[i & 1][a]);
        };
        load_all(0);
        load_all(1);
        if (w < EW) {
#pragma unroll
          for (int k = 0; k < KC; ++k) gc[k] = coh_ld1(gb, (size_t)max(st.cp[k], 0) * H + uj);
        }
        __builtin_amdgcn_sched_barrier(0);
        mul(0, 0, NGA, f[0]);
        load_all(2);
        __builtin_amdgcn_sched_barrier(0);
        mul(1, 0, NGA, f[1]);
        load_all(3);
        __builtin_amdgcn_sched_barrier(0);
        mul(2, 0, NGA, f[0]);
        mul(3, 0, NGA, f[1]);
      } else {
        Frag<BF> f0[3], g0[NCH];
#pragma unroll
        for (int a = 0; a < 3; ++a) load(0, a, f0[a]);
#pragma unroll
        for (int k = 0; k < NCH; ++k) load(0, 3 + k, g0[k]);
        if constexpr (CPW == 2) {
          Frag<BF> f1[3], g1[NCH];
#pragma unroll
          for (int a = 0; a < 3; ++a) load(1, a, f1[a]);
          if (w < EW) {
#pragma unroll
            for (int k = 0; k < KC; ++k)
              gc[k] = coh_ld1(gb, (size_t)max(st.cp[k], 0) * H + uj);
          }
          __builtin_amdgcn_sched_barrier(0);
          mul(0, 0, 3, f0);
          __builtin_amdgcn_sched_barrier(0);
          // the second chunk's f rows take the registers the first i|o|u freed
#pragma unroll
          for (int k = 0; k < NCH; ++k) load(1, 3 + k, g1[k]);
          __builtin_amdgcn_sched_barrier(0);
          mul(0, 3, NCH, g0);
          mul(1, 0, 3, f1);
          mul(1, 3, NCH, g1);
        } else {
          if (w < EW) {
#pragma unroll
            for (int k = 0; k < KC; ++k)
              gc[k] = coh_ld1(gb, (size_t)max(st.cp[k], 0) * H + uj);
          }
          mul(0, 0, 3, f0);
          mul(0, 3, NCH, g0);
        }
      }
#pragma unroll
      for (int q = 0; q < UT; ++q)
#pragma unroll
        for (int g = 0; g < NACC; ++g)
#pragma unroll
          for (int i = 0; i < 4; ++i) red[w][q * NACC + g][i][lane] = acc[q][g][i];
      __syncthreads();
      if (w < EW) {
        const int p = rows.pos(4 * gq + wr), j = uj;
        auto zsum = [&](int g) {
          float z = red[0][ut * NACC + g][wr][lane];
#pragma unroll
          for (int q = 1; q < KW; ++q) z += red[q][ut * NACC + g][wr][lane];
          return z;
        };
        const float zh = zsum(0);
        if constexpr (UT == 2) flush();   // an earlier tile of this level
#pragma unroll
        for (int k = 0; k < KC; ++k) {
          const int cp = p >= 0 ? st.cp[k] : -1;
          if (cp < 0) continue;
          const float ghp = NCH >= 2 ? zh + zsum(1 + kc0 + k) : zh;
          if (cp < n.fuse_from) {
            n.dHp[(size_t)cp * H + j] = ghp;
            continue;
          }
          const GatePre<NCH>& q = st.q[k];
          const float gh = ghp + q.lg, tau = tanh_(q.c);
          const float gcv = gc[k] + gh * q.og * (1.f - tau * tau);
          float* d = late.d[k];
          d[0] = gcv * q.ug * q.ig * (1.f - q.ig);
          d[2] = gh * tau * q.og * (1.f - q.og);
          d[3] = gcv * q.ig * (1.f - q.ug * q.ug);
#pragma unroll
          for (int e = 0; e < NCH; ++e) {
            float df = 0.f;
            if (q.cp[e] >= 0) {
              df = gcv * q.ck[e] * q.fk[e] * (1.f - q.fk[e]);
              n.dCp[(size_t)q.cp[e] * H + j] = gcv * q.fk[e];
            }
            d[e == 0 ? 1 : 3 + e] = df;
          }
          late.p[k] = cp;
          if constexpr (BF) {
#pragma unroll
            for (int g = 0; g < NGA; ++g) n.dAb[(size_t)cp * GW + g * H + j] = f2bf(d[g]);
          } else if (cp >= pbase) {
#pragma unroll
            for (int g = 0; g < NGA; ++g) store_parts(n, cp, g * H + j, d[g]);
          }
        }
      }
      if (w == KW - 1 && rt == 0 && t > t0) {
        xcd_level_list(xl, x, lm, l0, lst[cur ^ 1], &sm[cur ^ 1]);
      }
      if (16 * (rt + 1) < m) {
        if constexpr (UT == 1) flush();
        __syncthreads();
      }
    }
    if (t > t0) {
      if (m == 0) {   // nothing of this XCD yet: no barrier needed, only the next list
        if (w == KW - 1) xcd_level_list(xl, x, lm, l0, lst[cur ^ 1], &sm[cur ^ 1]);
        __syncthreads();
      } else {
        xcd_barrier_arrive(xl, s);
        flush();
      }
      l1 = l0;
      l0 = lm;
      lm = lmm;
      if (sm[cur ^ 1] > 0) fetch(ListRows{lst[cur ^ 1], sm[cur ^ 1], l0}, st);
      if (m > 0) xcd_barrier_wait(xl, s, nut);
    }
  }
  flush();
}

int xcd_mode() {
  const char* e = getenv("CAVS_XCD_LOOP");
  return e && e[0] ? (e[0] == '0' ? 0 : 1) : -1;
}

// The loop's suffix: the first level >= 1 from which every level has at most
// kXcdRows positions and that together hold no more positions than the owner kernel does (T: none).
int xcd_suffix(const int* lo_host, int T, int V) {
  int t = T;
  while (t > 1 && lo_host[t] - lo_host[t - 1] <= kXcdRows && V - lo_host[t - 1] <= kXcdMaxSuffix)
    --t;
  return t;
}

}  // namespace

// Weights in registers: 16 unit columns on each of an XCD's 32 CUs.  Three and
// four slots' operands fit beside them only with one chunk per wavefront.
// In bf16 a weight is one register instead of three: two unit tiles up to 1024
// (with two slots those spill, 25 registers forward and 39 backward, and still
// take a half of the level kernels' time on deep trees).  In fp32 the backward of
// two slots above 256 spills one, the others none.
bool xcd_applies(int H, int N, bool bf) { return H <= (N <= 2 ? (bf ? 1024 : 512) : 256); }

// By default from this many small levels on; CAVS_XCD_LOOP=1 takes the loop
// wherever it applies, =0 never.  The loop costs some 15 us to start (owners,
// weights, the grid's arrival), a training pass that twice, and saves more per
// level the wider the layer is.  us of a pass, loop minus level kernels, in
// batches of 3, 5, 7, 9 and 11 levels, the leaves' among them (chains and trees,
// 2 to 64 of them):
//   training   H = 64    +15 to 19,  +7 to 11,   -2 to 0,  -22 to -11,  -30 to -20
//              256       +13 to 17,  -2 to +7,  -16 to -3, -36 to -19,  -46 to -27
//              320, 512   +2 to 11, -22 to -3, -48 to -20, -74 to -36,  -96 to -54
//              bf16       -8 to 19, -43 to +9,  -76 to -6, -110 to -19, -144 to -32
//   inference  H = 64    +11 to 12,  +9 to 10,   +4 to 8,   +2 to 6,     0 to +4
//              256        +9 to 10,  +5 to 6,    0 to +3,   -5 to -2,   -10 to -8
//              320, 512   +8 to 13,  -2 to +5,  -14 to -2, -24 to -9,   -32 to -15
//              bf16       +3 to 14, -11 to 10,  -25 to +5, -39 to +1,   -52 to -5
// One line for both, so that inference sums in the training forward's order and
// its states are the same bit for bit: where a training pass gains more than an
// inference pass loses.
int xcd_min_levels(const Net& n) { return n.H <= 128 ? 8 : n.H <= 256 ? 6 : 5; }

int xcd_first_level(const Net& n, const int* lo_host, int T) {
  const int mode = xcd_mode();
  if (mode == 0 || !xcd_applies(n.H, n.N, n.bf)) return T;
  if ((size_t)n.V * n.GW >= (1u << 29)) return T;   // 32-bit offsets of the coherent loads
  const int t = xcd_suffix(lo_host, T, n.V);
  return mode < 0 && T - t < xcd_min_levels(n) ? T : t;
}

size_t xcd_ws_bytes(int V) { return (size_t)kXcdWords * 4 + (size_t)V; }

// rows of dA's split copy: the loop's suffix
size_t xcd_suffix_rows(const int* lo_host, int T, int V) {
  const int t = T > 1 ? xcd_suffix(lo_host, T, V) : T;
  return t < T ? (size_t)(V - lo_host[t]) : 0;
}

void xcd_owner(const Net& n, const int* lo_host, int t0, void* xws, hipStream_t s) {
  const int base = lo_host[t0];
  CAVS_LAUNCH("k_xcd_owner", k_xcd_owner, dim3(1), dim3(1024), 0, s, n.parent_pos, base,
              n.V - base, (unsigned char*)xws + (size_t)kXcdWords * 4, (int*)xws);
}

namespace {

struct LoopKernel {
  const void* fn;
  const char* name;
};

#define CAVS_LOOP(KIND, NCH, BF, CPW, UT)                                              \
  LoopKernel{reinterpret_cast<const void*>(&k_lstm_##KIND##_xcd<NCH, BF, CPW, UT>),    \
             "k_lstm_" #KIND "_xcd<" #NCH ", " #BF ", " #CPW ", " #UT ">"}
// one or two chunks per wavefront, or (bf16) four and two unit tiles
#define CAVS_LOOP_BF(KIND, NCH)                      \
  (n.H > 512   ? CAVS_LOOP(KIND, NCH, true, 4, 2)    \
   : n.H > 256 ? CAVS_LOOP(KIND, NCH, true, 2, 1)    \
               : CAVS_LOOP(KIND, NCH, true, 1, 1))
#define CAVS_LOOP_F32(KIND, NCH) \
  (n.H > 256 ? CAVS_LOOP(KIND, NCH, false, 2, 1) : CAVS_LOOP(KIND, NCH, false, 1, 1))
#define CAVS_LOOP_PICK(KIND)                                                 \
  (n.N == 4   ? CAVS_LOOP(KIND, 4, false, 1, 1)                              \
   : n.N == 3 ? CAVS_LOOP(KIND, 3, false, 1, 1)                              \
   : n.N == 2 ? (n.bf ? CAVS_LOOP_BF(KIND, 2) : CAVS_LOOP_F32(KIND, 2))      \
              : (n.bf ? CAVS_LOOP_BF(KIND, 1) : CAVS_LOOP_F32(KIND, 1)))

// The launch of the forward or backward loop over levels [t0, T); false when
// it cannot be launched.
bool xcd_launch(bool fwd, const Net& n, const int* lo, const int* lo_host, int t0, int T,
                void* xws, bool owner_ready, hipStream_t s) {
  if (t0 >= T) return true;
  int* words = (int*)xws;
  unsigned char* own = (unsigned char*)xws + (size_t)kXcdWords * 4;
  int dev = 0, ncu = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return false;
  const int G = ncu / 8 * 8;   // one workgroup per CU, the same number on every XCD
  const LoopKernel k = fwd ? CAVS_LOOP_PICK(fwd) : CAVS_LOOP_PICK(bwd);
  const int threads = 64 * kXcdKW;
  if (G / 8 * (n.H > 512 ? 32 : 16) < n.H ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k.fn, threads, 0) != hipSuccess || per < 1)
    return false;
  const LoopTurn turn(t_active_ctx->device, s);
  if (!turn.ok()) return false;
  if (!owner_ready) xcd_owner(n, lo_host, t0, xws, s);
  int spin = kXcdSpin;
  if (const char* e = getenv("CAVS_PERSIST_SPIN")) spin = atoi(e);
  XcdLoop xl{words, own, lo_host[t0], spin, t_active_ctx->dev_err_dev};
  int a0 = t0, a1 = T;
  void* args[] = {(void*)&n, (void*)&lo, (void*)&a0, (void*)&a1, (void*)&xl};
  TimedScope ts(k.name, s, lo_host[t0], lo_host[T] - lo_host[t0], /*bracket=*/true);
  // A plain launch: one workgroup per CU fits (checked above), the stream has
  // drained every earlier kernel of the library and the loops on other streams
  // are over (turn), so on a device shared with no other process all G
  // workgroups get to run.  The cooperative launch API guarantees no more than
  // that and measured about 15 us slower per launch.  Should another process
  // hold CUs, the workgroups that are resident wait, boundedly, for the rest; a
  // wait that gives up is reported through cavs_sync.
  return hipLaunchKernel(k.fn, dim3(G), dim3(threads), args, 0, s) == hipSuccess;
}

}  // namespace

bool lstm_fwd_xcd(const Net& n, const int* lo, const int* lo_host, int t0, int T, void* xws,
                  bool owner_ready, hipStream_t s) {
  return xcd_launch(true, n, lo, lo_host, t0, T, xws, owner_ready, s);
}

bool lstm_bwd_xcd(const Net& n, const int* lo, const int* lo_host, int t0, int T, void* xws,
                  bool owner_ready, hipStream_t s) {
  return xcd_launch(false, n, lo, lo_host, t0, T, xws, owner_ready, s);
}

}  // namespace cavs

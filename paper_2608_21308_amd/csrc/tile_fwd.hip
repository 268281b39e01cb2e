// Forward of the token-tiled path for long chunks (tile_common.h): Algorithm 1
// with one token kernel and one state kernel per chunk.
//
// Token kernel, key side (tile of 32 tokens, all hidden columns):
//   H = K W1^T, A = act(H), Y = A W2^T, dY from the LayerNorm of Y,
//   dA = dY W2, dH = dA act'(H); the operands of the token sums go to memory.
// Query side: O = Q + LN(act(Q W1^T) W2^T).
// State kernel: W <- cw W + cm M + sum_t K^W_t G_t, M <- cb M + sum_t K^M_t G_t.
// Operand precision is that of the chain kernels: W1 and the W2 of dA as bf16
// high and low parts, the MLP's first-layer sums over high and low parts of
// K_t dH (formed from the fp32 dH, which goes through memory whole), fp32
// accumulation and fp32 state.
#include <algorithm>

#include "tile_common.h"
#include "tile_path.h"

namespace e2ttt {

namespace {

template <class G>
struct FwdTileSmem {
  alignas(16) float red[2 * G::RED];
  alignas(16) Bf dy[G::TI];
  alignas(16) Bf it[3][G::IT];
  alignas(16) Bf tr[4][G::TR];
};

// Sum over the head index of the ring's next fragments (the bf16 high and low
// parts of each K-step in turn) with the token fragments.
template <class G, class RING>
__device__ __forceinline__ void first_layer(f32x4 (&h)[2], RING& ring, int n,
                                            const bf16x8 (&x)[2][G::KD]) {
  h[0] = zero4();
  h[1] = zero4();
#pragma unroll
  for (int p = 0; p < 2 * G::KD; ++p) {
    const bf16x8 wf = ring.take(n + p);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) h[tb] = mma8(h[tb], wf, x[tb][p >> 1]);
  }
}
// Y^T += W2 A^T over one block of 32 hidden columns.
template <class G, class RING>
__device__ __forceinline__ void second_layer(f32x4 (&y)[G::NIB][2], RING& ring, int n,
                                             const bf16x8& f0, const bf16x8& f1) {
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) {
    const bf16x8 wt = ring.take(n + ib);
    y[ib][0] = mma8(y[ib][0], wt, f0);
    y[ib][1] = mma8(y[ib][1], wt, f1);
  }
}
constexpr int kFwdRing = 16;
// Fragment sequence of the net at one side, per block q of 32 hidden columns:
// for both 16-column blocks each first-layer matrix (high, low per K-step),
// then the T fragments of W2.
template <class G>
struct NetSeq {
  static constexpr int PER = 2 * G::NF * 2 * G::KD + G::NIB;
  const bf16x8* rh;    // R copy, high part; the low part follows
  long copy16, t16;    // 16-byte vectors to the low part, to the T copy
  int dhb, w;
  __device__ __forceinline__ const bf16x8* operator()(int n) const {
    const int k = n / PER, e = n % PER;
    const int q = min(w + 4 * k, dhb - 1);
    constexpr int RB = G::NF * 2 * G::KD;      // R fragments of one 16-column block
    if (e < 2 * RB) {
      const int b = e / RB, m = e % RB / (2 * G::KD), p = e % (2 * G::KD);
      return rh + (p & 1) * copy16 + ((m * 2 * dhb + 2 * q + b) * G::KD + (p >> 1)) * 64;
    }
    return rh + t16 + ((G::SEC * G::NIB + (e - 2 * RB)) * dhb + q) * 64;
  }
};
// R fragments of the second-layer matrix (high, low per K-step).
template <class G>
struct DeltaSeq {
  static constexpr int PER = 2 * 2 * G::KD;
  const bf16x8* rh;
  long copy16;
  int dhb, w;
  __device__ __forceinline__ const bf16x8* operator()(int n) const {
    const int k = n / PER, e = n % PER, b = e / (2 * G::KD), p = e % (2 * G::KD);
    const int q = min(w + 4 * k, dhb - 1);
    return rh + (p & 1) * copy16 + ((G::SEC * 2 * dhb + 2 * q + b) * G::KD + (p >> 1)) * 64;
  }
};

// Per tile the whole of W1 high and low, W2 and its high and low parts pass from
// the L2 through the CU once, for 320 products a wave (dh 512, head dim 128).
// One workgroup per CU (306 registers); 62 us a launch at 32 units of 512 tokens
// with both sides (8.5 TB/s of operands), of which the matrix cores are busy 13 %
// and the VALU 30 %.
template <class G>
__device__ void fwd_key_tile(const TileFwdArgs& a, FwdTileSmem<G>& sm, long u, int tile, int len,
                             long row0) {
  constexpr int D = G::D, EPL = G::EPL, NF = G::NF;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, i0 = c * EPL;
  const int dhb = (a.dh + 31) / 32, njb = 2 * dhb;
  const bf16x8* const rh =
      reinterpret_cast<const bf16x8*>(a.wops + a.slot * a.wslot + u * a.wunit);
  char* const bop = a.bops + (u * a.ntile_max + tile) * (long)G::NB_FWD * njb * 1024;
  char* const aop = a.aops + (u * a.ntile_max + tile) * (long)G::NA_FWD * G::NIB * 1024;
  const Bf* kp = static_cast<const Bf*>(a.k) + row0 * D;
  const Bf* vp = static_cast<const Bf*>(a.v) + row0 * D;

  bf16x8 xf[2][G::KD];
  tok_frags<G>(xf, kp, len, g, c);
  f32x4 yacc[G::NIB][2];
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) yacc[ib][0] = yacc[ib][1] = zero4();
  using Seq = NetSeq<G>;
  FragRing<kFwdRing, Seq> ring(Seq{rh, a.copy / 16, a.toff / 16, dhb, w}, lane);
  f32x4 d1[NF][G::MAXQ][2][2];
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    const int q = w + 4 * k;
    if (q < dhb) {
      bf16x4 aq[2][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int jb = 2 * q + b;
        f32x4 h[NF][2];
#pragma unroll
        for (int m = 0; m < NF; ++m)
          first_layer<G>(h[m], ring, k * Seq::PER + (b * NF + m) * 2 * G::KD, xf);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          f32x4 act;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if constexpr (G::FW == 0) {
              const Act2 ga = gelu2(h[0][tb][r]);
              act[r] = ga.f;
              d1[0][k][b][tb][r] = ga.d1;
            } else {
              const float hg = h[0][tb][r], hu = h[NF - 1][tb][r], sg = sigm_f(hg);
              d1[NF - 1][k][b][tb][r] = hg * sg;
              d1[0][k][b][tb][r] = hu * sg * (1.0f + hg * (1.0f - sg));
              act[r] = hg * sg * hu;
            }
          }
          aq[b][tb] = cvt4(act);
        }
        st_frag(bop, (G::NB_FWD - 1) * njb + jb, lane,
                tr_tok<G>(sm.tr[w], aq[b][0], aq[b][1], g, c));
      }
      const bf16x8 f0 = join8(aq[0][0], aq[1][0]), f1 = join8(aq[0][1], aq[1][1]);
      second_layer<G>(yacc, ring, k * Seq::PER + 2 * NF * 2 * G::KD, f0, f1);
    }
  }
  reduce_waves<G>(yacc, sm.red, w, g, c);

  // LayerNorm and its backward, four rows per wave step, 16 lanes per row
  const float inv_d = 1.0f / D;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    const bool ok = t < len;
    float y[EPL], kv[EPL], vv[EPL], z[EPL], e[EPL], dy[EPL];
    red_row<G>(y, sm.red, t, i0);
    row_bf<EPL>(kv, kp + (long)t * D + i0, ok);
    row_bf<EPL>(vv, vp + (long)t * D + i0, ok);
    float sig = 1.0f;
    if (a.resln) {
      float s1 = 0.0f, s2 = 0.0f, se = 0.0f, sez = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) s1 += y[q];
      const float mu = group16_sum(s1) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { y[q] -= mu; s2 += y[q] * y[q]; }
      sig = rsq_f(group16_sum(s2) * inv_d + a.eps);   // 1 / sigma
      if (a.ln_a) {
        // f = k + a z + b: the LayerNorm backward takes a (v - f)
        float la[EPL], lb[EPL];
        row_f32<EPL>(la, a.ln_a + (u % a.H) * D + i0, true);
        row_f32<EPL>(lb, a.ln_b + (u % a.H) * D + i0, true);
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
          z[q] = y[q] * sig;
          e[q] = la[q] * (vv[q] - kv[q] - fmaf(la[q], z[q], lb[q]));
        }
      } else {
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
          z[q] = y[q] * sig;
          e[q] = vv[q] - kv[q] - z[q];
        }
      }
#pragma unroll
      for (int q = 0; q < EPL; ++q) { se += e[q]; sez += e[q] * z[q]; }
      const float me = group16_sum(se) * inv_d, mez = group16_sum(sez) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q) dy[q] = (e[q] - me - z[q] * mez) * sig;
    } else {
#pragma unroll
      for (int q = 0; q < EPL; ++q) { z[q] = y[q]; dy[q] = vv[q] - y[q]; }
    }
    if (a.zk && ok) {
      store_row_io<IoT<false>, EPL>(a.zk + (row0 + t) * D + i0, z);
      if (c == 0) st_stream(a.rk + row0 + t, sig);
    }
    const float kw = ok ? a.kw[row0 + t] : 0.0f, km = ok ? a.km[row0 + t] : 0.0f;
    put_ti<G>(sm.dy, t, i0, dy);
    put_it<G>(sm.it[0], t, i0, dy, kw);
    put_it<G>(sm.it[1], t, i0, dy, km);
    put_it<G>(sm.it[2], t, i0, kv);
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 3; ++x) flush_it<G>(aop + x * G::NIB * 1024, sm.it[x], w, lane, g, c);

  // dA = dY W2 and the first-layer deltas
  lds_tok_frags<G>(xf, sm.dy, g, c);
  using Seq2 = DeltaSeq<G>;
  FragRing<kFwdRing, Seq2> ring2(Seq2{rh, a.copy / 16, dhb, w}, lane);
  float kwt[2], kmt[2];
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const int t = 16 * tb + c;
    kwt[tb] = t < len ? a.kw[row0 + t] : 0.0f;
    kmt[tb] = t < len ? a.km[row0 + t] : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    const int q = w + 4 * k;
    if (q < dhb) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int jb = 2 * q + b;
        f32x4 da[2];
        first_layer<G>(da, ring2, k * Seq2::PER + b * 2 * G::KD, xf);
        if constexpr (G::FW == 0) {
          bf16x4 hi[2], lo[2];   // the halves of the fp32 words
#pragma unroll
          for (int tb = 0; tb < 2; ++tb)
            word_halves(da[tb] * d1[0][k][b][tb], hi[tb], lo[tb]);
          st_frag(bop, jb, lane, tr_tok<G>(sm.tr[w], hi[0], hi[1], g, c));
          st_frag(bop, njb + jb, lane, tr_tok<G>(sm.tr[w], lo[0], lo[1], g, c));
        } else {
#pragma unroll
          for (int m = 0; m < NF; ++m) {
            bf16x4 vw[2], vm[2];
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
              const f32x4 dh = da[tb] * d1[m][k][b][tb];
              vw[tb] = cvt4(kwt[tb] * dh);
              vm[tb] = cvt4(kmt[tb] * dh);
            }
            st_frag(bop, 2 * m * njb + jb, lane, tr_tok<G>(sm.tr[w], vw[0], vw[1], g, c));
            st_frag(bop, (2 * m + 1) * njb + jb, lane, tr_tok<G>(sm.tr[w], vm[0], vm[1], g, c));
          }
        }
      }
    }
  }
}

template <class G>
__device__ void fwd_query_tile(const TileFwdArgs& a, float* red, long u, int slot, int len,
                               long row0) {
  constexpr int D = G::D, EPL = G::EPL, NF = G::NF;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, i0 = c * EPL;
  const int dhb = (a.dh + 31) / 32;
  const bf16x8* const rh =
      reinterpret_cast<const bf16x8*>(a.wops + slot * a.wslot + u * a.wunit);
  const Bf* qp = static_cast<const Bf*>(a.q) + row0 * D;

  bf16x8 xf[2][G::KD];
  tok_frags<G>(xf, qp, len, g, c);
  f32x4 yacc[G::NIB][2];
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) yacc[ib][0] = yacc[ib][1] = zero4();
  using Seq = NetSeq<G>;
  FragRing<kFwdRing, Seq> ring(Seq{rh, a.copy / 16, a.toff / 16, dhb, w}, lane);
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    if (w + 4 * k >= dhb) break;
    bf16x4 aq[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      f32x4 h[NF][2];
#pragma unroll
      for (int m = 0; m < NF; ++m)
        first_layer<G>(h[m], ring, k * Seq::PER + (b * NF + m) * 2 * G::KD, xf);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        f32x4 act;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (G::FW == 0) act[r] = gelu_f(h[0][tb][r]);
          else act[r] = silu_f(h[0][tb][r]) * h[NF - 1][tb][r];
        }
        aq[b][tb] = cvt4(act);
      }
    }
    const bf16x8 f0 = join8(aq[0][0], aq[1][0]), f1 = join8(aq[0][1], aq[1][1]);
    second_layer<G>(yacc, ring, k * Seq::PER + 2 * NF * 2 * G::KD, f0, f1);
  }
  reduce_waves<G>(yacc, red, w, g, c);
  const float inv_d = 1.0f / D;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    const bool ok = t < len;
    float y[EPL], x[EPL], f[EPL];
    red_row<G>(y, red, t, i0);
    float sig = 1.0f;
    if (a.resln) {
      row_bf<EPL>(x, qp + (long)t * D + i0, ok);
      float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) s1 += y[q];
      const float mu = group16_sum(s1) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { y[q] -= mu; s2 += y[q] * y[q]; }
      sig = rsq_f(group16_sum(s2) * inv_d + a.eps);
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        y[q] *= sig;                                  // Z_Q
        f[q] = x[q] + y[q];
      }
      if (a.ln_a) {                                   // f = q + a Z_Q + b
        float la[EPL], lb[EPL];
        row_f32<EPL>(la, a.ln_a + (u % a.H) * D + i0, true);
        row_f32<EPL>(lb, a.ln_b + (u % a.H) * D + i0, true);
#pragma unroll
        for (int q = 0; q < EPL; ++q) f[q] = x[q] + fmaf(la[q], y[q], lb[q]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < EPL; ++q) f[q] = y[q];
    }
    if (ok) {
      store_row_io<IoT<true>, EPL>(static_cast<Bf*>(a.out) + (row0 + t) * D + i0, f);
      if (a.zq) {
        store_row_io<IoT<false>, EPL>(a.zq + (row0 + t) * D + i0, y);
        if (c == 0) st_stream(a.rq + row0 + t, sig);
      }
    }
  }
}

template <class G>
__global__ void __launch_bounds__(256, 1) tile_fwd_token_kernel(TileFwdArgs a) {
  __shared__ FwdTileSmem<G> sm;
  const TileBlock b = tile_block(blockIdx.x, a.U, 2 * a.ntile);
  if (b.u >= a.U) return;
  const bool key = b.item < a.ntile;     // the key side takes longer and goes first
  const int tile = key ? b.item : b.item - a.ntile;
  const int s0 = a.r * a.C + tile * kTileTok;
  const int len = min(kTileTok, min(a.T, (a.r + 1) * a.C) - s0);
  const long row0 = b.u * a.T + s0;
  if (key) fwd_key_tile<G>(a, sm, b.u, tile, len, row0);
  else fwd_query_tile<G>(a, sm.red, b.u, a.slot, len, row0);
}

// The query side alone, of chunks [r0, r0 + items / nt32) at once: what a chain
// launch that leaves it out runs behind itself (chain_fwd.hip).
template <class G>
__global__ void __launch_bounds__(256, 1) tile_fwd_query_kernel(TileFwdArgs a) {
  __shared__ __attribute__((aligned(16))) float red[2 * G::RED];
  const TileBlock b = tile_block(blockIdx.x, a.U, a.items);
  if (b.u >= a.U) return;
  const int r = a.r + b.item / a.ntile_max;
  const int s0 = r * a.C + b.item % a.ntile_max * kTileTok;
  const int len = min(kTileTok, min(a.T, (r + 1) * a.C) - s0);
  if (len <= 0) return;                  // past the end of a ragged chunk
  fwd_query_tile<G>(a, red, b.u, a.keep ? r : r - a.r, len, b.u * a.T + s0);
}

// Bound by memory: the B operands, the state in and out and its operand copies
// (about 150 MB a launch at 32 units of 512 tokens, head dim 128, dh 512: 35 us,
// 43 us while the state was read and written in the caller's layout).  The A
// operands of a tile, which the four waves share, are staged through LDS.
template <class G>
__global__ void __launch_bounds__(256, 1) tile_fwd_state_kernel(TileFwdArgs a) {
  constexpr int D = G::D, IH = G::IH, NMAT = G::NMAT, NF = G::NF, SEC = G::SEC;
  constexpr int NA = G::NA_FWD;
  constexpr int NV = (NA * IH * 64 + 255) / 256;   // staged 16-byte vectors per thread
  __shared__ __attribute__((aligned(16))) u32x4 sa[2][NA * IH * 64];
  __shared__ __attribute__((aligned(16))) float sk[2][2][kTileTok];
  __shared__ __attribute__((aligned(16))) Bf tr[4][4 * 20 * 4];
  const int dhb = (a.dh + 31) / 32, njb = 2 * dhb;
  const TileBlock blk = tile_block(blockIdx.x, a.U, (njb + 3) / 4 * 2);
  if (blk.u >= a.U) return;
  const long u = blk.u;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int ib0 = (blk.item & 1) * IH, jb = (blk.item >> 1) * 4 + w;
  const bool mine = jb < njb;                       // uniform over the wave
  const int j = 16 * jb + c;
  const bool okj = j < a.dh;
  const long dhd = (long)a.dh * D;
  auto off = [&](int m, int ib, int r) -> long {
    const int i = 16 * (ib0 + ib) + 4 * g + r;
    return m < SEC ? m * dhd + (long)j * D + i : SEC * dhd + (long)i * a.dh + j;
  };

  f32x4 W[NMAT][IH], M[NMAT][IH];
  // between chunks the state lies in register-tile order, one 16-byte vector
  // per lane and tile; the caller's arrays are read and written once
  f32x4* const st = reinterpret_cast<f32x4*>(a.state) + u * 2 * NMAT * njb * G::NIB * 64 + lane;
  auto at = [&](int x, int m, int ib) { return (((x * NMAT + m) * njb + jb) * G::NIB + ib0 + ib) * 64; };
  if (a.init) {
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
      for (int ib = 0; ib < IH; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          W[m][ib][r] = okj ? a.w_in[u * a.P + off(m, ib, r)] : 0.0f;
          M[m][ib][r] = (okj && a.m_in) ? a.m_in[u * a.P + off(m, ib, r)] : 0.0f;
        }
  } else {
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
      for (int ib = 0; ib < IH; ++ib) {
        W[m][ib] = mine ? st[at(0, m, ib)] : zero4();
        M[m][ib] = mine ? st[at(1, m, ib)] : zero4();
      }
  }

  if (!a.init) {
    const float* car = a.carry + (u * a.NC + a.r) * 3;
    const float cw = car[0], cm = car[1], cb = car[2];
    const int s0 = a.r * a.C, L = min(a.C, a.T - s0);
    const char* const aop = a.aops + u * a.ntile_max * (long)NA * G::NIB * 1024;
    const char* const bop = a.bops + u * a.ntile_max * (long)G::NB_FWD * njb * 1024;
    // B operands three tiles ahead, A operands and scalars two (one in flight,
    // one in LDS): a step is some 500 cycles, a load from memory several times that
    struct Stage {
      u32x4 v[NV];
      float k = 0.0f;
    } p0, p1;
    auto load_a = [&](Stage& p, int tile) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = tid + v * 256, x = e / (IH * 64), o = e % (IH * 64);
        if (e < NA * IH * 64)
          p.v[v] = reinterpret_cast<const u32x4*>(
              aop + ((long)tile * NA + x) * G::NIB * 1024)[ib0 * 64 + o];
      }
      const int t = tile * kTileTok + (tid & 31);
      if (tid < 64) p.k = t < L ? (tid < 32 ? a.kw : a.km)[u * a.T + s0 + t] : 0.0f;
    };
    using BFrags = bf16x8[G::NB_FWD];
    BFrags b0, b1, b2, b3;
    auto load_b = [&](BFrags& f, int tile) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int x = 0; x < G::NB_FWD; ++x)
        f[x] = ld_frag(bop + (long)tile * G::NB_FWD * njb * 1024, x * njb + (mine ? jb : 0), lane);
    };
    load_a(p0, 0);
    load_b(b0, 0);
    load_a(p1, 1);
    load_b(b1, 1);
    load_b(b2, 2);
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
      for (int ib = 0; ib < IH; ++ib) {
        W[m][ib] = cw * W[m][ib] + cm * M[m][ib];
        M[m][ib] = cb * M[m][ib];
      }
    // one tile: its staged operands to LDS, the loads of later tiles, the products
    auto step = [&](int tile, int par, Stage& p, const BFrags& f, BFrags& later) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (tid + v * 256 < NA * IH * 64) sa[par][tid + v * 256] = p.v[v];
      if (tid < 64) sk[par][tid >> 5][tid & 31] = p.k;
      __syncthreads();
      load_a(p, tile + 2);
      load_b(later, tile + 3);
      pin_loads();
      const bf16x8* sf = reinterpret_cast<const bf16x8*>(sa[par]);
      if constexpr (G::FW == 0) {
        // K^W_t dH and K^M_t dH as bf16 high and low parts
        bf16x4 wh[2], wl[2], mh[2], ml[2];
        const bf16x4 hh[2] = {__builtin_shufflevector(f[0], f[0], 0, 1, 2, 3),
                              __builtin_shufflevector(f[0], f[0], 4, 5, 6, 7)};
        const bf16x4 hl[2] = {__builtin_shufflevector(f[1], f[1], 0, 1, 2, 3),
                              __builtin_shufflevector(f[1], f[1], 4, 5, 6, 7)};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 x = from_halves(hh[h], hl[h]);
          const f32x4 vw = *reinterpret_cast<const f32x4*>(&sk[par][0][16 * h + 4 * g]) * x;
          const f32x4 vm = *reinterpret_cast<const f32x4*>(&sk[par][1][16 * h + 4 * g]) * x;
          wh[h] = cvt4(vw);
          wl[h] = cvt4(vw - quad_f32(wh[h]));
          mh[h] = cvt4(vm);
          ml[h] = cvt4(vm - quad_f32(mh[h]));
        }
        const bf16x8 fwh = join8(wh[0], wh[1]), fwl = join8(wl[0], wl[1]);
        const bf16x8 fmh = join8(mh[0], mh[1]), fml = join8(ml[0], ml[1]);
#pragma unroll
        for (int ib = 0; ib < IH; ++ib) {
          const bf16x8 yw = sf[ib * 64 + lane], ym = sf[(IH + ib) * 64 + lane];
          const bf16x8 kf = sf[(2 * IH + ib) * 64 + lane];
          W[SEC][ib] = mma8(W[SEC][ib], yw, f[2]);
          M[SEC][ib] = mma8(M[SEC][ib], ym, f[2]);
          W[0][ib] = mma8(W[0][ib], kf, fwh);
          M[0][ib] = mma8(M[0][ib], kf, fmh);
          W[0][ib] = mma8(W[0][ib], kf, fwl);
          M[0][ib] = mma8(M[0][ib], kf, fml);
        }
      } else {
#pragma unroll
        for (int ib = 0; ib < IH; ++ib) {
          const bf16x8 yw = sf[ib * 64 + lane], ym = sf[(IH + ib) * 64 + lane];
          const bf16x8 kf = sf[(2 * IH + ib) * 64 + lane];
          W[SEC][ib] = mma8(W[SEC][ib], yw, f[G::NB_FWD - 1]);
          M[SEC][ib] = mma8(M[SEC][ib], ym, f[G::NB_FWD - 1]);
#pragma unroll
          for (int m = 0; m < NF; ++m) {
            W[m][ib] = mma8(W[m][ib], kf, f[2 * m]);
            M[m][ib] = mma8(M[m][ib], kf, f[2 * m + 1]);
          }
        }
      }
    };
    // (a tile's buffers are rewritten two steps later, after the next step's barrier)
    for (int tile = 0; tile < a.ntile; tile += 4) {
      step(tile, 0, p0, b0, b3);
      step(tile + 1, 1, p1, b1, b0);
      step(tile + 2, 0, p0, b2, b1);
      step(tile + 3, 1, p1, b3, b2);
    }
  }

  if (mine) {
    if (a.last) {
      if (okj) {
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
#pragma unroll
          for (int ib = 0; ib < IH; ++ib)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              a.w_out[u * a.P + off(m, ib, r)] = W[m][ib][r];
              a.m_out[u * a.P + off(m, ib, r)] = M[m][ib][r];
            }
      }
    } else {
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
#pragma unroll
        for (int ib = 0; ib < IH; ++ib) {
          st[at(0, m, ib)] = W[m][ib];
          st[at(1, m, ib)] = M[m][ib];
        }
      char* const rh = a.wops + a.slot_next * a.wslot + u * a.wunit;
      char* const rl = rh + a.copy;
      char* const th = rl + a.copy;
      char* const mh = a.mops ? a.mops + a.slot_next * a.mslot + u * a.copy : nullptr;
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
#pragma unroll
        for (int p = 0; p < IH / 2; ++p) {
          const int fr = (m * njb + jb) * G::KD + ib0 / 2 + p;
          bf16x4 hi[2], lo[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            hi[h] = cvt4(W[m][2 * p + h]);
            lo[h] = cvt4(W[m][2 * p + h] - quad_f32(hi[h]));
            // T copy: the tile transposed through this wave's LDS
            *reinterpret_cast<bf16x4*>(&tr[w][(g * 20 + c) * 4]) = hi[h];
            wave_lds_order();
            const bf16x4 tq = ds_tr4(&tr[w][((c & 3) * 20 + 4 * g + (c >> 2)) * 4]);
            wave_lds_order();
            const int ib = ib0 + 2 * p + h;
            reinterpret_cast<bf16x4*>(
                th)[(((m * G::NIB + ib) * dhb + (jb >> 1)) * 64 + lane) * 2 + (jb & 1)] = tq;
          }
          st_frag(rh, fr, lane, join8(hi[0], hi[1]));
          st_frag(rl, fr, lane, join8(lo[0], lo[1]));
          if (mh) st_frag(mh, fr, lane, join8(cvt4(M[m][2 * p]), cvt4(M[m][2 * p + 1])));
        }
    }
  }
}

// The state kernel does not depend on the hidden blocks per wave.
template <class G>
using StateShape = TileShape<G::FW, G::D, 1>;

template <class G>
hipError_t run(const TileFwdArgs& base, hipStream_t s) {
  TileFwdArgs a = base;
  const long gs = tile_grid(a.U, tile_state_groups(a.dh));
  a.init = 1;
  a.slot_next = 0;
  hipLaunchKernelGGL(tile_fwd_state_kernel<StateShape<G>>, dim3((unsigned)gs), dim3(256), 0, s, a);
  a.init = 0;
  for (int r = 0; r < a.NC; ++r) {
    a.r = r;
    a.slot = a.keep ? r : 0;
    a.last = r + 1 == a.NC;
    a.slot_next = a.keep ? r + 1 : 0;
    a.ntile = (std::min(a.C, a.T - r * a.C) + kTileTok - 1) / kTileTok;
    hipLaunchKernelGGL(tile_fwd_token_kernel<G>, dim3((unsigned)tile_grid(a.U, 2 * a.ntile)),
                       dim3(256), 0, s, a);
    hipLaunchKernelGGL(tile_fwd_state_kernel<StateShape<G>>, dim3((unsigned)gs), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_fwd_query(const ChainConfig& cfg, TileFwdArgs a, int nchunks, hipStream_t s) {
  const int nq = ((a.dh + 31) / 32 + 3) / 4;
  a.items = nchunks * a.ntile_max;
  const dim3 grid((unsigned)tile_grid(a.U, a.items));
#define E2TTT_TILE(FW, D, MAXQ)                                                                \
  if (cfg.fw == FW && cfg.d == D && nq <= MAXQ) {                                              \
    hipLaunchKernelGGL((tile_fwd_query_kernel<TileShape<FW, D, MAXQ>>), grid, dim3(256), 0, s, \
                       a);                                                                     \
    return hipGetLastError();                                                                  \
  }
#include "tile_variants.inc"
#undef E2TTT_TILE
  return hipErrorInvalidValue;
}

hipError_t launch_tile_fwd(const ChainConfig& cfg, const TileFwdArgs& a, hipStream_t s) {
  const int nq = ((a.dh + 31) / 32 + 3) / 4;   // blocks of 32 hidden columns per wave
#define E2TTT_TILE(FW, D, MAXQ) \
  if (cfg.fw == FW && cfg.d == D && nq <= MAXQ) return run<TileShape<FW, D, MAXQ>>(a, s);
#include "tile_variants.inc"
#undef E2TTT_TILE
  return hipErrorInvalidValue;
}

}  // namespace e2ttt

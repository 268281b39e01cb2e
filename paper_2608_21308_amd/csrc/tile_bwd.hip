// Backward of the token-tiled path for long chunks (tile_common.h): reverse
// mode through the chunks, one token kernel and one state kernel per chunk,
// with the algebra of chain_bwd.hip (whose names are used here).
//
// Token kernel, key side, per tile of 32 tokens with all hidden columns:
//   pass 1 over the hidden columns: H, act and its derivatives recomputed from
//     the chunk-start weights, u = K Wb1^T, K Mb1^T, r = dY Wb2, dY Mb2, the
//     scalar-kernel adjoints, dAh, Hh without its Yh term, and the sums over j
//     dk += dH (K^W Wb1 + K^M Mb1), dYh = A (K^W Wb2 + K^M Mb2)^T + dAh W2^T;
//   the second-order LayerNorm step (eh, Yh, dv);
//   pass 2: Hh += (Yh W2) act'(H), dk += Hh W1.
// Query side: Yb_Q, Hb_Q and dq.  Both leave the operands of the state sums.
// State kernel: Mb <- cm Wb + cb Mb, Wb <- cw Wb + the sums over the tokens,
// the carry adjoints before it, and the operand copies for the next chunk.
//
// The factors K^W_t, K^M_t go onto the activations before they are rounded to
// bf16 (one rounding, as for the unscaled ones), so that the products with Wb
// and Mb share one accumulator.
#include <algorithm>

#include "tile_common.h"
#include "tile_path.h"

namespace e2ttt {

namespace {

template <class G>
struct BwdQuerySmem {
  alignas(16) float red[2 * G::RED];       // also the K^T buffer of the first row phase
  alignas(16) Bf xt[G::TI];                // K | Q
  alignas(16) Bf ti[G::TI];                // dY, then Yh | Yb_Q
  alignas(16) Bf it[G::IT];                // dY^T, then Yh^T | Yb_Q^T
  alignas(16) Bf tr[4][G::TR];
};
template <class G>
struct BwdTileSmem : BwdQuerySmem<G> {
  // Hh of pass 1, one f32x4 per lane, matrix, 16-column block and token block
  alignas(16) f32x4 hh[G::NF * G::MAXQ * 4 * 256];
  float kb[2][4][kTileTok];                // dK^W, dK^M partials of the waves
};

// e = a (v - f) (or v - f), z and 1/sigma of one row at the saved LayerNorm output.
template <class G>
struct KeyRow {
  float z[G::EPL], e[G::EPL], kv[G::EPL];
  float sig, me, mez;
  __device__ __forceinline__ void load(const TileBwdArgs& a, long u, long row, int i0, bool ok) {
    constexpr int EPL = G::EPL, D = G::D;
    const float inv_d = 1.0f / D;
    float v[EPL];
    row_bf<EPL>(kv, static_cast<const Bf*>(a.k) + row * D + i0, ok);
    row_bf<EPL>(v, static_cast<const Bf*>(a.v) + row * D + i0, ok);
    row_f32<EPL>(z, a.zk + row * D + i0, ok);
    if (a.resln) {
      sig = ok ? a.rk[row] : 0.0f;
      if (a.ln_a) {
        float la[EPL], lb[EPL];
        row_f32<EPL>(la, a.ln_a + (u % a.H) * D + i0, true);
        row_f32<EPL>(lb, a.ln_b + (u % a.H) * D + i0, true);
#pragma unroll
        for (int q = 0; q < EPL; ++q) e[q] = la[q] * (v[q] - kv[q] - fmaf(la[q], z[q], lb[q]));
      } else {
#pragma unroll
        for (int q = 0; q < EPL; ++q) e[q] = v[q] - kv[q] - z[q];
      }
      float se = 0.0f, sez = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { se += e[q]; sez += e[q] * z[q]; }
      me = group16_sum(se) * inv_d;
      mez = group16_sum(sez) * inv_d;
    } else {
      sig = 1.0f;
      me = mez = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { e[q] = v[q] - z[q]; z[q] = 0.0f; }
    }
  }
  // dY of the row
  __device__ __forceinline__ void delta(float (&dy)[G::EPL]) const {
#pragma unroll
    for (int q = 0; q < G::EPL; ++q) dy[q] = (e[q] - me - z[q] * mez) * sig;
  }
};

// acc (rows i, columns t) += the ring's next T fragments (one K-step over the
// hidden index) times the B fragments.
template <class G, class RING>
__device__ __forceinline__ void hidden_sum(f32x4 (&acc)[G::NIB][2], RING& ring, int n,
                                           const bf16x8& f0, const bf16x8& f1) {
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) {
    const bf16x8 wt = ring.take(n + ib);
    acc[ib][0] = mma8(acc[ib][0], wt, f0);
    acc[ib][1] = mma8(acc[ib][1], wt, f1);
  }
}
// N products over the head index with one token operand (a [t][i] LDS array),
// from the ring's next R fragments (K-step by K-step, the N operands in turn).
template <class G, int N, class RING>
__device__ __forceinline__ void head_sums(f32x4 (&r)[N][2], RING& ring, int n, const Bf* x, int g,
                                          int c) {
#pragma unroll
  for (int p = 0; p < G::KD; ++p) {
    bf16x8 xf[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      const Bf* xp = x + (16 * tb + c) * G::LDD + 32 * p + 4 * g;
      xf[tb] = join8(*reinterpret_cast<const bf16x4*>(xp),
                     *reinterpret_cast<const bf16x4*>(xp + 16));
    }
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const bf16x8 wf = ring.take(n + p * N + m);
      r[m][0] = mma8(r[m][0], wf, xf[0]);
      r[m][1] = mma8(r[m][1], wf, xf[1]);
    }
  }
}
template <class G>
constexpr int kBwdRing = G::FW == 0 ? 16 : 12;
// Fragment sequence of pass 1, per block q of 32 hidden columns: for both
// 16-column blocks the R fragments of W_0, Wb, Mb of the first-layer matrices,
// then of the second, K-step by K-step; then the T
// fragments of Wb, Mb of the first-layer matrices, of Wb, Mb, W_0 of the second.
template <class G>
struct KeySeq {
  static constexpr int RB = 3 * G::NMAT * G::KD;      // R fragments of a 16-column block
  static constexpr int PER = 2 * RB + (2 * G::NF + 3) * G::NIB;
  const bf16x8* w0;    // R copy of W_0 (T copy two copies on)
  const bf16x8* gb;    // R of Wb, T of Wb, R of Mb, T of Mb
  long copy16;
  int dhb, w;
  __device__ __forceinline__ const bf16x8* operator()(int n) const {
    const int k = n / PER, e = n % PER;
    const int q = min(w + 4 * k, dhb - 1);
    if (e < 2 * RB) {
      const int b = e / RB, f = e % RB;
      const bool first = f < 3 * G::NF * G::KD;
      const int f2 = first ? f : f - 3 * G::NF * G::KD, x = f2 % 3;
      const int p = first ? f2 / (3 * G::NF) : f2 / 3;
      const int m = first ? f2 / 3 % G::NF : G::SEC;
      const bf16x8* base = x == 0 ? w0 : gb + (x == 1 ? 0 : 2 * copy16);
      return base + ((m * 2 * dhb + 2 * q + b) * G::KD + p) * 64;
    }
    const int t = (e - 2 * RB) / G::NIB, ib = (e - 2 * RB) % G::NIB;
    const int m = t < 2 * G::NF ? t / 2 : G::SEC;
    const bf16x8* base = t == 2 * G::NF + 2 ? w0 + 2 * copy16
                                            : gb + ((t & 1) == 0 ? copy16 : 3 * copy16);
    return base + ((m * G::NIB + ib) * dhb + q) * 64;
  }
};
// Pass 2: R fragments of W2 for both 16-column blocks, T fragments of the first layer.
template <class G>
struct HessSeq {
  static constexpr int PER = 2 * G::KD + G::NF * G::NIB;
  const bf16x8* w0;
  long copy16;
  int dhb, w;
  __device__ __forceinline__ const bf16x8* operator()(int n) const {
    const int k = n / PER, e = n % PER;
    const int q = min(w + 4 * k, dhb - 1);
    if (e < 2 * G::KD)
      return w0 + ((G::SEC * 2 * dhb + 2 * q + e / G::KD) * G::KD + e % G::KD) * 64;
    const int m = (e - 2 * G::KD) / G::NIB, ib = (e - 2 * G::KD) % G::NIB;
    return w0 + 2 * copy16 + ((m * G::NIB + ib) * dhb + q) * 64;
  }
};
// Query side, per 16-column block: R fragments of the first layer (MLP: its low
// part too), of W2; then the T fragments of the first layer.
template <class G>
struct QuerySeq {
  static constexpr int NR = G::FW == 0 ? 2 : G::NF;   // first-layer R groups of a block
  static constexpr int RB = (NR + 1) * G::KD;
  static constexpr int PER = 2 * RB + G::NF * G::NIB;
  const bf16x8* w0;
  long copy16;
  int dhb, w;
  __device__ __forceinline__ const bf16x8* operator()(int n) const {
    const int k = n / PER, e = n % PER;
    const int q = min(w + 4 * k, dhb - 1);
    if (e < 2 * RB) {
      const int b = e / RB, f = e % RB;
      const bool first = f < NR * G::KD;
      const int x = first ? f % NR : NR, p = first ? f / NR : f - NR * G::KD;
      const int m = !first ? G::SEC : (G::FW == 0 ? 0 : x);
      const bf16x8* base = w0 + (G::FW == 0 && x == 1 ? copy16 : 0);
      return base + ((m * 2 * dhb + 2 * q + b) * G::KD + p) * 64;
    }
    const int m = (e - 2 * RB) / G::NIB, ib = (e - 2 * RB) % G::NIB;
    return w0 + 2 * copy16 + ((m * G::NIB + ib) * dhb + q) * 64;
  }
};

// Thirteen copies of a matrix pass from the L2 through the CU per tile (MLP), for
// some 700 products a wave at dh 512, head dim 128; 440 registers, one workgroup
// per CU.  120 us a launch at 32 units of 512 tokens with the query side
// (10 TB/s of operands).
template <class G>
__device__ void bwd_key_tile(const TileBwdArgs& a, BwdTileSmem<G>& sm, long u, int tile, int len,
                             long row0) {
  constexpr int D = G::D, EPL = G::EPL, NF = G::NF;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, c = lane & 15, i0 = c * EPL;
  const int dhb = (a.dh + 31) / 32, njb = 2 * dhb;
  const bf16x8* const w0 =
      reinterpret_cast<const bf16x8*>(a.wops + a.r * a.wslot + u * a.wunit);
  const bf16x8* const gb = reinterpret_cast<const bf16x8*>(a.gops + u * 4 * a.copy);
  char* const bop = a.bops + (u * a.ntile_max + tile) * (long)G::NB_KEY * njb * 1024;
  char* const aop = a.aops + (u * a.ntile_max + tile) * (long)G::NA_KEY * G::NIB * 1024;
  const float inv_d = 1.0f / D;
  constexpr int AOP = G::NIB * 1024;

  // first-order rows: dY, and the operands dY^T, K^T of the state sums
  Bf* const kt = reinterpret_cast<Bf*>(sm.red);
  static_assert(G::IT * 2 <= 2 * G::RED * 4, "the K^T buffer fits the partial-sum buffers");
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    KeyRow<G> x;
    x.load(a, u, row0 + (t < len ? t : 0), i0, t < len);
    float dy[EPL];
    x.delta(dy);
    put_ti<G>(sm.ti, t, i0, dy);
    put_it<G>(sm.it, t, i0, dy);
    put_it<G>(kt, t, i0, x.kv);
    put_ti<G>(sm.xt, t, i0, x.kv);
  }
  __syncthreads();
  flush_it<G>(aop, sm.it, w, lane, g, c);
  flush_it<G>(aop + 2 * AOP, kt, w, lane, g, c);

  float kw[2], km[2], kwp[2] = {0.0f, 0.0f}, kmp[2] = {0.0f, 0.0f};
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const int t = 16 * tb + c;
    kw[tb] = t < len ? a.kw[row0 + t] : 0.0f;
    km[tb] = t < len ? a.km[row0 + t] : 0.0f;
  }
  f32x4 dk[G::NIB][2], dyh[G::NIB][2];
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) dk[ib][0] = dk[ib][1] = dyh[ib][0] = dyh[ib][1] = zero4();
  f32x4 d1[NF][G::MAXQ][2][2];
  using Seq = KeySeq<G>;
  FragRing<kBwdRing<G>, Seq> ring(Seq{w0, gb, a.copy / 16, dhb, w}, lane);
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    const int q = w + 4 * k;
    if (q < dhb) {
      bf16x4 hw[NF][2][2], hm[NF][2][2], aw[2][2], am[2][2], ah[2][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int jb = 2 * q + b;
        // of each first-layer matrix H, u with Wb, u with Mb; dA, r with Wb, with Mb
        f32x4 hu3[3 * NF][2], yr[3][2];
#pragma unroll
        for (int x = 0; x < 3 * NF; ++x) hu3[x][0] = hu3[x][1] = zero4();
#pragma unroll
        for (int x = 0; x < 3; ++x) yr[x][0] = yr[x][1] = zero4();
        const int nb = k * Seq::PER + b * Seq::RB;
        head_sums<G, 3 * NF>(hu3, ring, nb, sm.xt, g, c);
        head_sums<G, 3>(yr, ring, nb + 3 * NF * G::KD, sm.ti, g, c);
        bf16x4 aq[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          f32x4 dh[NF], dah, hh[NF], af;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float r2 = kw[tb] * yr[1][tb][r] + km[tb] * yr[2][tb][r];
            if constexpr (G::FW == 0) {
              const Act3 ga = gelu3(hu3[0][tb][r]);
              af[r] = ga.f;
              d1[0][k][b][tb][r] = ga.d1;
              dh[0][r] = yr[0][tb][r] * ga.d1;
              const float pp = kw[tb] * hu3[1][tb][r] + km[tb] * hu3[2][tb][r];
              dah[r] = pp * ga.d1;
              hh[0][r] = pp * yr[0][tb][r] * ga.d2 + r2 * ga.d1;
              kwp[tb] += dh[0][r] * hu3[1][tb][r] + af[r] * yr[1][tb][r];
              kmp[tb] += dh[0][r] * hu3[2][tb][r] + af[r] * yr[2][tb][r];
            } else {
              constexpr int M1 = NF - 1;
              const float hg = hu3[0][tb][r], hu = hu3[3 * M1][tb][r];
              const Act3 sa = silu3(hg);
              af[r] = sa.f * hu;
              d1[0][k][b][tb][r] = hu * sa.d1;
              d1[M1][k][b][tb][r] = sa.f;
              dh[0][r] = yr[0][tb][r] * hu * sa.d1;
              dh[M1][r] = yr[0][tb][r] * sa.f;
              const float pg = kw[tb] * hu3[1][tb][r] + km[tb] * hu3[2][tb][r];
              const float pu = kw[tb] * hu3[3 * M1 + 1][tb][r] + km[tb] * hu3[3 * M1 + 2][tb][r];
              dah[r] = pg * hu * sa.d1 + pu * sa.f;
              hh[0][r] = pg * yr[0][tb][r] * hu * sa.d2 + pu * yr[0][tb][r] * sa.d1 + r2 * hu * sa.d1;
              hh[M1][r] = pg * yr[0][tb][r] * sa.d1 + r2 * sa.f;
              kwp[tb] += dh[0][r] * hu3[1][tb][r] + dh[M1][r] * hu3[3 * M1 + 1][tb][r] + af[r] * yr[1][tb][r];
              kmp[tb] += dh[0][r] * hu3[2][tb][r] + dh[M1][r] * hu3[3 * M1 + 2][tb][r] + af[r] * yr[2][tb][r];
            }
          }
#pragma unroll
          for (int m = 0; m < NF; ++m) {
            sm.hh[(((m * G::MAXQ + k) * 2 + b) * 2 + tb) * 256 + tid] = hh[m];
            hw[m][b][tb] = cvt4(kw[tb] * dh[m]);
            hm[m][b][tb] = cvt4(km[tb] * dh[m]);
          }
          aw[b][tb] = cvt4(kw[tb] * af);
          am[b][tb] = cvt4(km[tb] * af);
          ah[b][tb] = cvt4(dah);
          aq[tb] = cvt4(af);
        }
        st_frag(bop, jb, lane, tr_tok<G>(sm.tr[w], aq[0], aq[1], g, c));
        st_frag(bop, njb + jb, lane, tr_tok<G>(sm.tr[w], ah[b][0], ah[b][1], g, c));
      }
      const int nt = k * Seq::PER + 2 * Seq::RB;
#pragma unroll
      for (int m = 0; m < NF; ++m) {
        hidden_sum<G>(dk, ring, nt + 2 * m * G::NIB, join8(hw[m][0][0], hw[m][1][0]),
                      join8(hw[m][0][1], hw[m][1][1]));
        hidden_sum<G>(dk, ring, nt + (2 * m + 1) * G::NIB, join8(hm[m][0][0], hm[m][1][0]),
                      join8(hm[m][0][1], hm[m][1][1]));
      }
      hidden_sum<G>(dyh, ring, nt + 2 * NF * G::NIB, join8(aw[0][0], aw[1][0]),
                    join8(aw[0][1], aw[1][1]));
      hidden_sum<G>(dyh, ring, nt + (2 * NF + 1) * G::NIB, join8(am[0][0], am[1][0]),
                    join8(am[0][1], am[1][1]));
      hidden_sum<G>(dyh, ring, nt + (2 * NF + 2) * G::NIB, join8(ah[0][0], ah[1][0]),
                    join8(ah[0][1], ah[1][1]));
    }
  }
  // dK^W, dK^M of the tile's tokens: over the lane groups here, over the waves below
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    kwp[tb] += __shfl_xor(kwp[tb], 16);
    kwp[tb] += __shfl_xor(kwp[tb], 32);
    kmp[tb] += __shfl_xor(kmp[tb], 16);
    kmp[tb] += __shfl_xor(kmp[tb], 32);
    if (g == 0) {
      sm.kb[0][w][16 * tb + c] = kwp[tb];
      sm.kb[1][w][16 * tb + c] = kmp[tb];
    }
  }
  __syncthreads();   // every wave has flushed K^T from the partial-sum buffers
  reduce_waves<G>(dyh, sm.red, w, g, c);
  if (tid < 2 * kTileTok) {
    const int x = tid / kTileTok, t = tid % kTileTok;
    if (t < len)
      (x == 0 ? a.kwb : a.kmb)[row0 + t] =
          (sm.kb[x][0][t] + sm.kb[x][1][t]) + (sm.kb[x][2][t] + sm.kb[x][3][t]);
  }

  // LayerNorm second order
  float ehr[2][EPL];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    const bool ok = t < len;
    float d[EPL], yh[EPL];
    red_row<G>(d, sm.red, t, i0);
    float(&eh)[EPL] = ehr[s];
    if (a.resln) {
      KeyRow<G> x;
      x.load(a, u, row0 + (ok ? t : 0), i0, ok);
      float dy[EPL], zh[EPL];
      x.delta(dy);
      float m1 = 0.0f, m2 = 0.0f, sdd = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { m1 += d[q]; m2 += d[q] * x.z[q]; }
      m1 = group16_sum(m1) * inv_d;
      m2 = group16_sum(m2) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        eh[q] = (d[q] - m1 - x.z[q] * m2) * x.sig;
        sdd += d[q] * dy[q];
      }
      const float sh = -group16_sum(sdd) * x.sig;
#pragma unroll
      for (int q = 0; q < EPL; ++q) zh[q] = -(d[q] * x.mez + x.e[q] * m2) * x.sig;
      if (a.ln_a) {
        // f = k + a z + b: e's adjoint is a eh, z takes -a^2 eh; eh itself (the
        // adjoint of a e) is kept for the affine's gradients
        float la[EPL];
        row_f32<EPL>(la, a.ln_a + (u % a.H) * D + i0, true);
        if (ok) store_row_io<IoT<false>, EPL>(a.ln_zbar + (row0 + t) * D + i0, eh);
#pragma unroll
        for (int q = 0; q < EPL; ++q) {
          zh[q] -= la[q] * la[q] * eh[q];
          eh[q] *= la[q];
        }
      } else {
#pragma unroll
        for (int q = 0; q < EPL; ++q) zh[q] -= eh[q];
      }
      float n1 = 0.0f, n2 = 0.0f;
#pragma unroll
      for (int q = 0; q < EPL; ++q) { n1 += zh[q]; n2 += zh[q] * x.z[q]; }
      n1 = group16_sum(n1) * inv_d;
      n2 = group16_sum(n2) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q)
        yh[q] = (zh[q] - n1 - x.z[q] * n2) * x.sig + sh * x.z[q] * inv_d;
    } else {
#pragma unroll
      for (int q = 0; q < EPL; ++q) { eh[q] = d[q]; yh[q] = -d[q]; }
    }
    if (ok) store_row_io<IoT<true>, EPL>(static_cast<Bf*>(a.dv) + (row0 + t) * D + i0, eh);
    put_ti<G>(sm.ti, t, i0, yh);
    put_it<G>(sm.it, t, i0, yh);
  }
  __syncthreads();
  flush_it<G>(aop + AOP, sm.it, w, lane, g, c);

  // pass 2
  using Seq2 = HessSeq<G>;
  FragRing<kBwdRing<G>, Seq2> ring2(Seq2{w0, a.copy / 16, dhb, w}, lane);
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    const int q = w + 4 * k;
    if (q < dhb) {
      bf16x4 hq[NF][2][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int jb = 2 * q + b;
        f32x4 y2[1][2] = {{zero4(), zero4()}};
        head_sums<G, 1>(y2, ring2, k * Seq2::PER + b * G::KD, sm.ti, g, c);
#pragma unroll
        for (int m = 0; m < NF; ++m) {
#pragma unroll
          for (int tb = 0; tb < 2; ++tb)
            hq[m][b][tb] = cvt4(sm.hh[(((m * G::MAXQ + k) * 2 + b) * 2 + tb) * 256 + tid] +
                                y2[0][tb] * d1[m][k][b][tb]);
          st_frag(bop, (2 + m) * njb + jb, lane,
                  tr_tok<G>(sm.tr[w], hq[m][b][0], hq[m][b][1], g, c));
        }
      }
#pragma unroll
      for (int m = 0; m < NF; ++m)
        hidden_sum<G>(dk, ring2, k * Seq2::PER + 2 * G::KD + m * G::NIB,
                      join8(hq[m][0][0], hq[m][1][0]), join8(hq[m][0][1], hq[m][1][1]));
    }
  }
  reduce_waves<G>(dk, sm.red, w, g, c);   // (its buffers were read before the barrier above)
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    float d[EPL];
    red_row<G>(d, sm.red, t, i0);
    if (a.resln) {
#pragma unroll
      for (int q = 0; q < EPL; ++q) d[q] -= ehr[s][q];
    }
    if (t < len) store_row_io<IoT<true>, EPL>(static_cast<Bf*>(a.dk) + (row0 + t) * D + i0, d);
  }
}

template <class G>
__device__ void bwd_query_tile(const TileBwdArgs& a, BwdQuerySmem<G>& sm, long u, int chunk,
                               int len, long row0, char* aop, char* bop) {
  constexpr int D = G::D, EPL = G::EPL, NF = G::NF;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, i0 = c * EPL;
  const int dhb = (a.dh + 31) / 32, njb = 2 * dhb;
  const bf16x8* const w0 =
      reinterpret_cast<const bf16x8*>(a.wops + chunk * a.wslot + u * a.wunit);
  const float inv_d = 1.0f / D;
  constexpr int AOP = G::NIB * 1024;
  const Bf* qp = static_cast<const Bf*>(a.q) + row0 * D;
  const Bf* op = static_cast<const Bf*>(a.d_out) + row0 * D;

  Bf* const qt = reinterpret_cast<Bf*>(sm.red);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    const bool ok = t < len;
    float x[EPL], yb[EPL];
    row_bf<EPL>(yb, op + (long)t * D + i0, ok);
    row_bf<EPL>(x, qp + (long)t * D + i0, ok);
    if (a.resln) {   // LayerNorm backward of dO (a dO with the affine)
      const float sig = ok ? a.rq[row0 + t] : 0.0f;
      float z[EPL], m1 = 0.0f, m2 = 0.0f;
      row_f32<EPL>(z, a.zq + (row0 + t) * D + i0, ok);
      if (a.ln_a) {
        float la[EPL];
        row_f32<EPL>(la, a.ln_a + (u % a.H) * D + i0, true);
#pragma unroll
        for (int q = 0; q < EPL; ++q) yb[q] *= la[q];
      }
#pragma unroll
      for (int q = 0; q < EPL; ++q) { m1 += yb[q]; m2 += yb[q] * z[q]; }
      m1 = group16_sum(m1) * inv_d;
      m2 = group16_sum(m2) * inv_d;
#pragma unroll
      for (int q = 0; q < EPL; ++q) yb[q] = (yb[q] - m1 - z[q] * m2) * sig;
    }
    put_ti<G>(sm.ti, t, i0, yb);
    put_it<G>(sm.it, t, i0, yb);
    put_it<G>(qt, t, i0, x);
    put_ti<G>(sm.xt, t, i0, x);
  }
  __syncthreads();
  flush_it<G>(aop, sm.it, w, lane, g, c);
  flush_it<G>(aop + AOP, qt, w, lane, g, c);
  f32x4 dq[G::NIB][2];
#pragma unroll
  for (int ib = 0; ib < G::NIB; ++ib) dq[ib][0] = dq[ib][1] = zero4();
  using Seq = QuerySeq<G>;
  FragRing<kBwdRing<G>, Seq> ring(Seq{w0, a.copy / 16, dhb, w}, lane);
#pragma unroll
  for (int k = 0; k < G::MAXQ; ++k) {
    const int q = w + 4 * k;
    if (q >= dhb) break;
    bf16x4 hb[NF][2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int jb = 2 * q + b;
      f32x4 hr[Seq::NR][2], ab[1][2] = {{zero4(), zero4()}};
#pragma unroll
      for (int x = 0; x < Seq::NR; ++x) hr[x][0] = hr[x][1] = zero4();
      const int nb = k * Seq::PER + b * Seq::RB;
      head_sums<G, Seq::NR>(hr, ring, nb, sm.xt, g, c);
      head_sums<G, 1>(ab, ring, nb + Seq::NR * G::KD, sm.ti, g, c);
      // the MLP's query side takes W_0's low part too, as the forward did
      if constexpr (G::FW == 0) {
        hr[0][0] += hr[1][0];
        hr[0][1] += hr[1][1];
      }
      bf16x4 aq[2];
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        f32x4 act, d1[NF];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (G::FW == 0) {
            const Act2 ga = gelu2(hr[0][tb][r]);
            act[r] = ga.f;
            d1[0][r] = ga.d1;
          } else {
            const float hg = hr[0][tb][r], hu = hr[NF - 1][tb][r], sg = sigm_f(hg);
            d1[NF - 1][r] = hg * sg;
            d1[0][r] = hu * sg * (1.0f + hg * (1.0f - sg));
            act[r] = hg * sg * hu;
          }
        }
        aq[tb] = cvt4(act);
#pragma unroll
        for (int m = 0; m < NF; ++m) hb[m][b][tb] = cvt4(ab[0][tb] * d1[m]);
      }
      st_frag(bop, jb, lane, tr_tok<G>(sm.tr[w], aq[0], aq[1], g, c));
#pragma unroll
      for (int m = 0; m < NF; ++m)
        st_frag(bop, (1 + m) * njb + jb, lane,
                tr_tok<G>(sm.tr[w], hb[m][b][0], hb[m][b][1], g, c));
    }
#pragma unroll
    for (int m = 0; m < NF; ++m)
      hidden_sum<G>(dq, ring, k * Seq::PER + 2 * Seq::RB + m * G::NIB,
                    join8(hb[m][0][0], hb[m][1][0]), join8(hb[m][0][1], hb[m][1][1]));
  }
  __syncthreads();   // every wave has flushed Q^T from the partial-sum buffers
  reduce_waves<G>(dq, sm.red, w, g, c);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int t = 16 * s + 4 * w + g;
    if (t < len) {
      float d[EPL];
      red_row<G>(d, sm.red, t, i0);
      if (a.resln) {
        float x[EPL];
        row_bf<EPL>(x, op + (long)t * D + i0, true);
#pragma unroll
        for (int q = 0; q < EPL; ++q) d[q] += x[q];
      }
      store_row_io<IoT<true>, EPL>(static_cast<Bf*>(a.dq) + (row0 + t) * D + i0, d);
    }
  }
}

template <class G>
__global__ void __launch_bounds__(256, 1) tile_bwd_token_kernel(TileBwdArgs a) {
  __shared__ BwdTileSmem<G> sm;
  static_assert(sizeof(BwdTileSmem<G>) <= 160 * 1024, "LDS budget");
  const TileBlock b = tile_block(blockIdx.x, a.U, 2 * a.ntile);
  if (b.u >= a.U) return;
  const bool key = b.item < a.ntile;     // the key side takes longer and goes first
  const int tile = key ? b.item : b.item - a.ntile;
  const int s0 = a.r * a.C + tile * kTileTok;
  const int len = min(kTileTok, min(a.T, (a.r + 1) * a.C) - s0);
  const long row0 = b.u * a.T + s0;
  if (key) bwd_key_tile<G>(a, sm, b.u, tile, len, row0);
  else {
    const long t = b.u * a.ntile_max + tile;
    const int njb = (a.dh + 31) / 32 * 2;
    bwd_query_tile<G>(a, sm, b.u, a.r, len, row0, a.qaops + t * (G::NA_QRY * G::NIB * 1024),
                      a.qbops + t * (G::NB_QRY * njb * 1024L));
  }
}

// The query side alone, of every chunk at once: none of it depends on the
// adjoint state.  Ahead of a chain that leaves it out (chain_bwd.hip, QOFF).  (Not
// ahead of the token kernels: with up to 128 tiles a chunk their query sides run
// beside the key sides at no cost, and a launch of their own made the backward's
// training step 2 to 14 % slower; with more tiles it gained 2 to 4 %, for memory
// that grows with the sequence.)
template <class G>
__global__ void __launch_bounds__(256, 1) tile_bwd_query_kernel(TileBwdArgs a) {
  __shared__ BwdQuerySmem<G> sm;
  const TileBlock b = tile_block(blockIdx.x, a.U, a.NC * a.ntile_max);
  if (b.u >= a.U) return;
  const int r = b.item / a.ntile_max, tile = b.item % a.ntile_max;
  const int s0 = r * a.C + tile * kTileTok;
  const int len = min(kTileTok, min(a.T, (r + 1) * a.C) - s0);
  if (len <= 0) return;                  // past the end of a ragged chunk
  const long t = (b.u * a.NC + r) * a.ntile_max + tile;
  const int njb = (a.dh + 31) / 32 * 2;
  bwd_query_tile<G>(a, sm, b.u, r, len, b.u * a.T + s0,
                    a.qaops + t * (G::NA_QRY * G::NIB * 1024),
                    a.qbops + t * (G::NB_QRY * njb * 1024L));
}

// Bound by memory as the forward's.  Two workgroups per CU where their registers
// allow it: 40 us at 32 units of 512 tokens, head dim 128, dh 512 (one workgroup
// of 380 registers: 67 us).
template <class G>
__global__ void __launch_bounds__(256, G::FW == 0 || G::D == 64 ? 2 : 1)
    tile_bwd_state_kernel(TileBwdArgs a) {
  constexpr int D = G::D, IH = G::IH, NMAT = G::NMAT, NF = G::NF, SEC = G::SEC;
  constexpr int NA = G::NA_KEY + G::NA_QRY, NB = G::NB_KEY + G::NB_QRY;
  constexpr int BD = G::FW == 0 && D == 64 ? 3 : 1;
  constexpr int NV = (NA * IH * 64 + 255) / 256;   // staged 16-byte vectors per thread
  static_assert(NA * IH * 64 % 64 == 0, "whole waves of vectors");
  __shared__ __attribute__((aligned(16))) u32x4 sa[2][NA * IH * 64];
  __shared__ __attribute__((aligned(16))) Bf tr[4][4 * 20 * 4];
  __shared__ float sc[4][3];
  const int dhb = (a.dh + 31) / 32, njb = 2 * dhb;
  const int items = (njb + 3) / 4 * 2;
  const TileBlock blk = tile_block(blockIdx.x, a.U, items);
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
          W[m][ib][r] = (okj && a.d_w_out) ? a.d_w_out[u * a.P + off(m, ib, r)] : 0.0f;
          M[m][ib][r] = (okj && a.d_m_out) ? a.d_m_out[u * a.P + off(m, ib, r)] : 0.0f;
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
    const long tk = u * a.ntile_max;                            // the chunk's tiles
    // B operands BD tiles ahead (as many as two workgroups per CU leave
    // registers for), A operands two (one in flight, one in LDS)
    struct Stage {
      u32x4 v[NV];
    } p0, p1;
    auto load_a = [&](Stage& p, int tile) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = tid + v * 256, x = e / (IH * 64), o = e % (IH * 64);
        const char* src = x < G::NA_KEY
                              ? a.aops + ((tk + tile) * G::NA_KEY + x) * (G::NIB * 1024)
                              : a.qaops + ((tk + tile) * G::NA_QRY + x - G::NA_KEY) * (G::NIB * 1024);
        if (e < NA * IH * 64) p.v[v] = reinterpret_cast<const u32x4*>(src)[ib0 * 64 + o];
      }
    };
    using BFrags = bf16x8[NB];
    BFrags b0, b1, b2, b3;
    auto load_b = [&](BFrags& f, int tile) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const char* src = x < G::NB_KEY
                              ? a.bops + ((tk + tile) * G::NB_KEY + x) * (njb * 1024L)
                              : a.qbops + ((tk + tile) * G::NB_QRY + x - G::NB_KEY) * (njb * 1024L);
        f[x] = ld_frag(src, mine ? jb : 0, lane);
      }
    };
    load_a(p0, 0);
    load_b(b0, 0);
    load_a(p1, 1);
    if constexpr (BD == 3) {
      load_b(b1, 1);
      load_b(b2, 2);
    }
    // carry adjoints <Wb, W_0>, <Wb, M_0>, <Mb, M_0> of this workgroup's share
    {
      const char* const w0 = a.wops + a.r * a.wslot + u * a.wunit;
      const char* const m0 = a.mops + a.r * a.mslot + u * a.copy;
      float pcw = 0.0f, pcm = 0.0f, pcb = 0.0f;
      if (mine) {
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
#pragma unroll
          for (int p = 0; p < IH / 2; ++p) {
            const int fr = (m * njb + jb) * G::KD + ib0 / 2 + p;
            const bf16x8 wf = ld_frag(w0, fr, lane), mf = ld_frag(m0, fr, lane);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float wv = (float)wf[4 * h + r], mv = (float)mf[4 * h + r];
                pcw += W[m][2 * p + h][r] * wv;
                pcm += W[m][2 * p + h][r] * mv;
                pcb += M[m][2 * p + h][r] * mv;
              }
          }
      }
      pcw = wave_sum(pcw);
      pcm = wave_sum(pcm);
      pcb = wave_sum(pcb);
      if (lane == 0) { sc[w][0] = pcw; sc[w][1] = pcm; sc[w][2] = pcb; }
    }
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
      for (int ib = 0; ib < IH; ++ib) {
        const f32x4 wb = W[m][ib];
        M[m][ib] = cm * wb + cb * M[m][ib];
        W[m][ib] = cw * wb;
      }
    // one tile: its staged operands to LDS, the loads of later tiles, the products
    auto step = [&](int tile, int par, Stage& p, const BFrags& f, BFrags& later) {
      if (tile >= a.ntile) return;
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (tid + v * 256 < NA * IH * 64) sa[par][tid + v * 256] = p.v[v];
      __syncthreads();
      load_a(p, tile + 2);
      load_b(later, tile + BD);
      pin_loads();
      const bf16x8* sf = reinterpret_cast<const bf16x8*>(sa[par]);
      auto ao = [&](int x, int ib) { return sf[(x * IH + ib) * 64 + lane]; };
#pragma unroll
      for (int ib = 0; ib < IH; ++ib) {
        W[SEC][ib] = mma8(W[SEC][ib], ao(0, ib), f[1]);        // dY^T dAh
        W[SEC][ib] = mma8(W[SEC][ib], ao(1, ib), f[0]);        // Yh^T A
        W[SEC][ib] = mma8(W[SEC][ib], ao(3, ib), f[2 + NF]);   // Yb_Q^T A_Q
        const bf16x8 kf = ao(2, ib), qf = ao(4, ib);
#pragma unroll
        for (int m = 0; m < NF; ++m) {
          W[m][ib] = mma8(W[m][ib], kf, f[2 + m]);             // K^T Hh
          W[m][ib] = mma8(W[m][ib], qf, f[3 + NF + m]);        // Q^T Hb_Q
        }
      }
    };
    // (a tile's buffers are rewritten two steps later, after the next step's barrier)
    if constexpr (BD == 3) {
      for (int tile = 0; tile < a.ntile; tile += 4) {
        step(tile, 0, p0, b0, b3);
        step(tile + 1, 1, p1, b1, b0);
        step(tile + 2, 0, p0, b2, b1);
        step(tile + 3, 1, p1, b3, b2);
      }
    } else {
      for (int tile = 0; tile < a.ntile; tile += 2) {
        step(tile, 0, p0, b0, b1);
        step(tile + 1, 1, p1, b1, b0);
      }
    }
    if (tid < 3)
      a.carryb[(((long)blk.item * a.U + u) * a.NC + a.r) * 3 + tid] =
          (sc[0][tid] + sc[1][tid]) + (sc[2][tid] + sc[3][tid]);
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
              a.d_w_in[u * a.P + off(m, ib, r)] = W[m][ib][r];
              a.d_m_in[u * a.P + off(m, ib, r)] = M[m][ib][r];
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
      char* const base = a.gops + u * 4 * a.copy;
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        char* const rc = base + 2 * x * a.copy;
        char* const tc = rc + a.copy;
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
#pragma unroll
          for (int p = 0; p < IH / 2; ++p) {
            bf16x4 hi[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              hi[h] = cvt4(x == 0 ? W[m][2 * p + h] : M[m][2 * p + h]);
              // T copy: the tile transposed through this wave's LDS
              *reinterpret_cast<bf16x4*>(&tr[w][(g * 20 + c) * 4]) = hi[h];
              wave_lds_order();
              const bf16x4 tq = ds_tr4(&tr[w][((c & 3) * 20 + 4 * g + (c >> 2)) * 4]);
              wave_lds_order();
              const int ib = ib0 + 2 * p + h;
              reinterpret_cast<bf16x4*>(
                  tc)[(((m * G::NIB + ib) * dhb + (jb >> 1)) * 64 + lane) * 2 + (jb & 1)] = tq;
            }
            st_frag(rc, (m * njb + jb) * G::KD + ib0 / 2 + p, lane, join8(hi[0], hi[1]));
          }
      }
    }
  }
}

// The state kernel does not depend on the hidden blocks per wave.
template <class G>
using StateShape = TileShape<G::FW, G::D, 1>;

template <class G>
hipError_t run(const TileBwdArgs& base, hipStream_t s) {
  TileBwdArgs a = base;
  const long gs = tile_grid(a.U, tile_state_groups(a.dh));
  a.init = 1;
  a.last = 0;
  a.r = a.NC - 1;
  hipLaunchKernelGGL(tile_bwd_state_kernel<StateShape<G>>, dim3((unsigned)gs), dim3(256), 0, s, a);
  a.init = 0;
  for (int r = a.NC - 1; r >= 0; --r) {
    a.r = r;
    a.last = r == 0;
    a.ntile = (std::min(a.C, a.T - r * a.C) + kTileTok - 1) / kTileTok;
    hipLaunchKernelGGL(tile_bwd_token_kernel<G>,
                       dim3((unsigned)tile_grid(a.U, 2 * a.ntile)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(tile_bwd_state_kernel<StateShape<G>>, dim3((unsigned)gs), dim3(256), 0, s,
                       a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_bwd_query(const ChainConfig& cfg, const TileBwdArgs& a, hipStream_t s) {
  const int nq = ((a.dh + 31) / 32 + 3) / 4;
  const dim3 grid((unsigned)tile_grid(a.U, a.NC * a.ntile_max));
#define E2TTT_TILE(FW, D, MAXQ)                                                                \
  if (cfg.fw == FW && cfg.d == D && nq <= MAXQ) {                                              \
    hipLaunchKernelGGL((tile_bwd_query_kernel<TileShape<FW, D, MAXQ>>), grid, dim3(256), 0, s, \
                       a);                                                                     \
    return hipGetLastError();                                                                  \
  }
#include "tile_variants.inc"
#undef E2TTT_TILE
  return hipErrorInvalidValue;
}

hipError_t launch_tile_bwd(const ChainConfig& cfg, const TileBwdArgs& a, hipStream_t s) {
  const int nq = ((a.dh + 31) / 32 + 3) / 4;   // blocks of 32 hidden columns per wave
#define E2TTT_TILE(FW, D, MAXQ) \
  if (cfg.fw == FW && cfg.d == D && nq <= MAXQ) return run<TileShape<FW, D, MAXQ>>(a, s);
#include "tile_variants.inc"
#undef E2TTT_TILE
  return hipErrorInvalidValue;
}

bool tile_supported(const ChainConfig& cfg, int dh) {
  const int nq = ((dh + 31) / 32 + 3) / 4;
#define E2TTT_TILE(FW, D, MAXQ) \
  if (cfg.bf && cfg.fw == FW && cfg.d == D && nq <= MAXQ) return true;
#include "tile_variants.inc"
#undef E2TTT_TILE
  return false;
}

int tile_state_groups(int dh) { return ((dh + 31) / 32 * 2 + 3) / 4 * 2; }

long tile_aop_bytes(const ChainConfig& cfg, TileOps ops) {
  using G = TileShape<0, 64, 1>;
  const long n = ops == kTileFwd ? G::NA_FWD : (ops == kTileBwdKey ? G::NA_KEY : G::NA_QRY);
  return n * (cfg.d / 16) * 1024;
}

long tile_bop_bytes(const ChainConfig& cfg, int dh, TileOps ops) {
  using G0 = TileShape<0, 64, 1>;
  using G1 = TileShape<1, 64, 1>;
  const bool sw = cfg.fw != 0;
  const long n = ops == kTileFwd      ? (sw ? G1::NB_FWD : G0::NB_FWD)
                 : ops == kTileBwdKey ? (sw ? G1::NB_KEY : G0::NB_KEY)
                                      : (sw ? G1::NB_QRY : G0::NB_QRY);
  return n * ((dh + 31) / 32 * 2) * 1024;
}

}  // namespace e2ttt

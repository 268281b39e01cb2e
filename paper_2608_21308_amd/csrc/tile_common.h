// Token-tiled path for long chunks: shapes, operand layouts and helpers shared
// by tile_fwd.hip and tile_bwd.hip.
//
// All tokens of a chunk take their gradients and outputs at the chunk-start
// weights, so inside a chunk the token tiles are independent.  Per chunk this
// path runs two launches:
//   a token kernel  one workgroup per (unit, 32-token tile, key or query side),
//                   holding the whole hidden width, so that the contractions
//                   over the hidden index end inside the workgroup;
//   a state kernel  one workgroup per (unit, 64 hidden columns, half of the
//                   head index): the sums over the chunk's tokens, the
//                   transition of the state, and the operand copies of the new
//                   state for the next chunk's token kernel.
// The chain kernels instead split a unit's hidden columns over workgroups and
// swap partial sums once per tile; with eight ranks at head dim 128 that swap
// and the sums over ranks were most of a tile's time.  Training step, chain
// then tiles: 32 units of 2048 tokens, head dim 128, dh 512, C = 512: 2.62 ms,
// 1.06 ms; 16 units of 1500 tokens, SwiGLU dh 344: 2.40 ms, 0.50 ms.
//
// Everything that a matrix instruction reads from memory lies there in
// fragment order, 16 bytes per lane, one wave-wide load per fragment:
//   R copies of a matrix   fragment (jb, p): lane 16 g + c holds
//                          W(i = 32 p + 16 h + 4 g + r, j = 16 jb + c), h < 2, r < 4
//                          (contraction over the head index i)
//   T copies of a matrix   fragment (ib, q): lane holds
//                          W(i = 16 ib + c, j = 32 q + 16 h + 4 g + r)
//                          (contraction over the hidden index j)
//   A operands of a tile   fragment ib: x(t = 16 h + 4 g + r, i = 16 ib + c)
//   B operands of a tile   fragment jb: x(t = 16 h + 4 g + r, j = 16 jb + c)
//                          (contraction over the tile's 32 tokens t)
// The token kernels form transposed tiles (rows j, columns t): a lane's four
// accumulator values are then consecutive hidden indices of one token, which
// is the operand quad of the contraction over j that follows, so activations
// go from one product to the next in registers.  Each of the four waves takes
// every fourth block of 32 hidden columns and keeps its own sums over them;
// the four partial sums meet once per tile in LDS, in wave order.
#pragma once

#include "chain_common.h"
#include "tile_path.h"

namespace e2ttt {

template <int FW_, int D_, int MAXQ_>
struct TileShape {
  static constexpr int FW = FW_;
  static constexpr int D = D_;
  static constexpr int MAXQ = MAXQ_;             // blocks of 32 hidden columns per wave
  static constexpr int NMAT = FW == 0 ? 2 : 3;
  static constexpr int NF = NMAT - 1;            // first-layer matrices
  static constexpr int SEC = NMAT - 1;           // the second-layer matrix
  static constexpr int NIB = D / 16;
  static constexpr int KD = D / 32;              // K-steps over the head index
  static constexpr int EPL = D / 16;             // head elements per lane in row phases
  static constexpr int IH = NIB / 2;             // 16-row head blocks of one state workgroup
  static constexpr int LDD = D + 4;              // [t][i] operand rows (bf16)
  static constexpr int LDR = D + 4;              // [t][i] partial-sum rows (fp32)
  static constexpr int LDT = kTileTok + 4;       // quad rows of the transposing buffers
  // B operands of a tile: forward MLP dH (fp32, its upper and its lower 16 bits
  // as two fragments, so that both transpose as bf16 ones do), A; SwiGLU
  // K^W dH and K^M dH of both matrices, A; backward key side A, dAh, Hh, query
  // side A_Q, Hb_Q
  static constexpr int NB_FWD = FW == 0 ? 3 : 5;
  static constexpr int NB_KEY = 2 + NF;
  static constexpr int NB_QRY = 1 + NF;
  static constexpr int NA_FWD = 3;               // K^W dY, K^M dY, K
  static constexpr int NA_KEY = 3;               // dY, Yh, K
  static constexpr int NA_QRY = 2;               // Yb_Q, Q
  static constexpr int RED = kTileTok * LDR;     // floats of one partial-sum buffer
  static constexpr int TI = kTileTok * LDD;      // elements of a [t][i] operand
  static constexpr int IT = (D / 4) * LDT * 4;   // elements of an [i][t] quad buffer
  static constexpr int TR = 4 * LDT * 4;         // elements of one wave's transposing buffer
};

typedef __bf16 Bf;

// Workgroup -> (unit, item).  With eight units or more, all items of a unit
// run on one XCD (workgroups are dealt to the XCDs round-robin), whose L2 then
// holds that unit's operand copies; with fewer the items spread over all.
struct TileBlock {
  long u;
  int item;
};
__host__ __device__ inline long tile_grid(long U, int items) {
  return U >= 8 ? 8 * ((U + 7) / 8) * items : U * items;
}
__device__ __forceinline__ TileBlock tile_block(long b, long U, int items) {
  TileBlock r;
  if (U >= 8) {
    const long s = b >> 3;
    r.u = (b & 7) + 8 * (s / items);
    r.item = (int)(s % items);
  } else {
    r.u = b / items;
    r.item = (int)(b % items);
  }
  return r;
}

__device__ __forceinline__ bf16x8 ld_frag(const void* base, int idx, int lane) {
  return reinterpret_cast<const bf16x8*>(base)[idx * 64 + lane];
}
__device__ __forceinline__ f32x4 mma8(f32x4 acc, const bf16x8& a, const bf16x8& b) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 join8(const bf16x4& a, const bf16x4& b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ bf16x4 cvt4(const f32x4& x) { return OpT<true>::cvt(x); }

// The upper and lower 16 bits of four fp32 words, and back.
__device__ __forceinline__ void word_halves(const f32x4& x, bf16x4& hi, bf16x4& lo) {
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  const s16x8 w = __builtin_bit_cast(s16x8, x);
  hi = __builtin_bit_cast(bf16x4, __builtin_shufflevector(w, w, 1, 3, 5, 7));
  lo = __builtin_bit_cast(bf16x4, __builtin_shufflevector(w, w, 0, 2, 4, 6));
}
__device__ __forceinline__ f32x4 from_halves(const bf16x4& hi, const bf16x4& lo) {
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  return __builtin_bit_cast(f32x4, __builtin_shufflevector(__builtin_bit_cast(s16x4, lo),
                                                           __builtin_bit_cast(s16x4, hi), 0, 4, 1,
                                                           5, 2, 6, 3, 7));
}

// One transposing LDS read: within each group of 16 lanes, lane c receives
// element c mod 4 of the quads addressed by lanes 4 r + c / 4, r = 0..3.
__device__ __forceinline__ bf16x4 ds_tr4(const Bf* p) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s4* lds_s4;
  return __builtin_bit_cast(bf16x4,
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4) const_cast<Bf*>(p)));
}
// LDS written and read by the same wave: its LDS operations complete in order;
// this only keeps the compiler from exchanging them.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Fragment of 16-row block blk over 32 contraction indices of a quad buffer
// (quad (4 blk + row quad) LD + k holds four rows at contraction index k).
template <int LD>
__device__ __forceinline__ bf16x8 quad_frag(const Bf* buf, int blk, int g, int c) {
  const Bf* p = buf + ((4 * blk + (c & 3)) * LD + 4 * g + (c >> 2)) * 4;
  return join8(ds_tr4(p), ds_tr4(p + 16 * 4));
}
// The transposed tile held as quads (rows j = 4 g .. of tokens 16 tb + c) of
// one 16-column block, as the B-operand fragment over the 32 tokens.
template <class G>
__device__ __forceinline__ bf16x8 tr_tok(Bf* buf, const bf16x4& t0, const bf16x4& t1, int g,
                                         int c) {
  *reinterpret_cast<bf16x4*>(buf + (g * G::LDT + c) * 4) = t0;
  *reinterpret_cast<bf16x4*>(buf + (g * G::LDT + 16 + c) * 4) = t1;
  wave_lds_order();
  const bf16x8 f = quad_frag<G::LDT>(buf, 0, g, c);
  wave_lds_order();
  return f;
}
__device__ __forceinline__ void st_frag(void* base, int idx, int lane, const bf16x8& f) {
  reinterpret_cast<bf16x8*>(base)[idx * 64 + lane] = f;
}

// Token-tile fragments over the head index from a row-major global tensor
// (column t = 16 tb + c, rows beyond len read as zero).
template <class G>
__device__ __forceinline__ void tok_frags(bf16x8 (&f)[2][G::KD], const Bf* rows, int len, int g,
                                          int c) {
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const int t = 16 * tb + c;
    const Bf* p = rows + (long)(t < len ? t : 0) * G::D + 4 * g;
#pragma unroll
    for (int k = 0; k < G::KD; ++k) {
      bf16x4 a = *reinterpret_cast<const bf16x4*>(p + 32 * k);
      bf16x4 b = *reinterpret_cast<const bf16x4*>(p + 32 * k + 16);
      if (t >= len) {
        a = cvt4(zero4());
        b = a;
      }
      f[tb][k] = join8(a, b);
    }
  }
}
// The same from a [t][i] LDS operand.
template <class G>
__device__ __forceinline__ void lds_tok_frags(bf16x8 (&f)[2][G::KD], const Bf* ti, int g, int c) {
#pragma unroll
  for (int tb = 0; tb < 2; ++tb)
#pragma unroll
    for (int k = 0; k < G::KD; ++k) {
      const Bf* p = ti + (16 * tb + c) * G::LDD + 32 * k + 4 * g;
      f[tb][k] = join8(*reinterpret_cast<const bf16x4*>(p),
                       *reinterpret_cast<const bf16x4*>(p + 16));
    }
}

// EPL consecutive bf16 / fp32 values of a row (zero when !ok).
template <int EPL>
__device__ __forceinline__ void row_bf(float (&x)[EPL], const Bf* p, bool ok) {
  if (ok) {
#pragma unroll
    for (int k = 0; k < EPL / 4; ++k) {
      const f32x4 v = quad_f32(reinterpret_cast<const bf16x4*>(p)[k]);
#pragma unroll
      for (int q = 0; q < 4; ++q) x[4 * k + q] = v[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < EPL; ++q) x[q] = 0.0f;
  }
}
template <int EPL>
__device__ __forceinline__ void row_f32(float (&x)[EPL], const float* p, bool ok) {
  if (ok) {
#pragma unroll
    for (int k = 0; k < EPL / 4; ++k) {
      const f32x4 v = reinterpret_cast<const f32x4*>(p)[k];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[4 * k + q] = v[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < EPL; ++q) x[q] = 0.0f;
  }
}
// EPL consecutive head indices of token t into a [t][i] operand / into an
// [i][t] quad buffer (scaled), one 8-byte store per four.
template <class G>
__device__ __forceinline__ void put_ti(Bf* dst, int t, int i0, const float (&v)[G::EPL]) {
#pragma unroll
  for (int k = 0; k < G::EPL / 4; ++k)
    *reinterpret_cast<bf16x4*>(dst + t * G::LDD + i0 + 4 * k) =
        cvt4(f32x4{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]});
}
template <class G>
__device__ __forceinline__ void put_it(Bf* dst, int t, int i0, const float (&v)[G::EPL],
                                       float s = 1.0f) {
#pragma unroll
  for (int k = 0; k < G::EPL / 4; ++k)
    *reinterpret_cast<bf16x4*>(dst + ((i0 / 4 + k) * G::LDT + t) * 4) =
        cvt4(f32x4{s * v[4 * k], s * v[4 * k + 1], s * v[4 * k + 2], s * v[4 * k + 3]});
}
// The A-operand fragments of an [i][t] quad buffer to global memory (wave w
// takes every fourth head block).
template <class G>
__device__ __forceinline__ void flush_it(void* dst, const Bf* it, int w, int lane, int g, int c) {
#pragma unroll
  for (int ib = w; ib < G::NIB; ib += 4) st_frag(dst, ib, lane, quad_frag<G::LDT>(it, ib, g, c));
}

// Partial sums of the four waves (transposed tiles: lane (g, c) holds head
// indices 16 ib + 4 g .. of token 16 tb + c): afterwards the sum is
// red[0][t][i] + red[1][t][i], (wave 0 + wave 2) + (wave 1 + wave 3).
// Ends in a barrier; begins with one when the buffers may still be read.
template <class G>
__device__ __forceinline__ void reduce_waves(f32x4 (&acc)[G::NIB][2], float* red, int w, int g,
                                             int c) {
  float* mine = red + (w & 1) * G::RED + c * G::LDR + 4 * g;
  if (w >= 2) {
#pragma unroll
    for (int ib = 0; ib < G::NIB; ++ib)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
        *reinterpret_cast<f32x4*>(mine + 16 * tb * G::LDR + 16 * ib) = acc[ib][tb];
  }
  __syncthreads();
  if (w < 2) {
#pragma unroll
    for (int ib = 0; ib < G::NIB; ++ib)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        f32x4* p = reinterpret_cast<f32x4*>(mine + 16 * tb * G::LDR + 16 * ib);
        *p = acc[ib][tb] + *p;
      }
  }
  __syncthreads();
}
template <class G>
__device__ __forceinline__ void red_row(float (&y)[G::EPL], const float* red, int t, int i0) {
#pragma unroll
  for (int q = 0; q < G::EPL; ++q)
    y[q] = red[t * G::LDR + i0 + q] + red[G::RED + t * G::LDR + i0 + q];
}

// Keeps loads from memory and matrix instructions on their side of this point
// (between loads alone, the scheduler gathers the products ahead of the loads).
__device__ __forceinline__ void pin_loads() { __builtin_amdgcn_sched_barrier(0x7C6); }

// Matrix operands arrive R loads ahead of their use: a wave has one to two
// thousand cycles of L2 latency to cover and nobody to take its place (one or
// two waves per SIMD), and left to itself the compiler issues a fragment's
// load just ahead of its product (measured at 32 units of 512 tokens, head dim
// 128, dh 512: the backward token kernel 275 us that way, 120 us with the ring).
// SRC maps the
// running number of a fragment to its address; a wave's sequence is fixed at
// compile time, so ring positions are registers.  Numbers past the end must
// map to a readable address.
template <int R, class SRC>
struct FragRing {
  bf16x8 f[R];
  SRC src;         // uniform addresses
  unsigned off;    // this lane's byte offset in a fragment
  __device__ __forceinline__ bf16x8 load(int n) const {
    return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(src(n)) + off);
  }
  __device__ __forceinline__ FragRing(SRC s, int lane) : src(s), off(16u * (unsigned)lane) {
#pragma unroll
    for (int i = 0; i < R; ++i) f[i] = load(i);
    pin_loads();
  }
  __device__ __forceinline__ bf16x8 take(int n) {
    const bf16x8 r = f[n % R];
    f[n % R] = load(n + R);
    pin_loads();
    return r;
  }
};

}  // namespace e2ttt

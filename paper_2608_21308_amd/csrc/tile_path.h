// Arguments and launchers of the token-tiled path (tile_common.h).
#pragma once

#include "e2ttt_internal.h"

namespace e2ttt {

constexpr int kTileTok = 32;   // tokens of a tile (one K-step of the state sums)

struct TileFwdArgs {
  const void* q;
  const void* k;
  const void* v;
  const float* kw;      // [U][T]
  const float* km;
  const float* carry;   // [U][NC][3]
  const float* w_in;
  const float* m_in;    // nullable
  float* state;         // [U][W | M] running state, fp32 in register-tile order
  void* out;
  float* w_out;
  float* m_out;
  char* wops;           // [slot][U][R high | R low | T] copies of W
  char* mops;           // [slot][U][R] copies of M (saving only, else null)
  char* aops;           // [U][ntile_max][NA][NIB] A operands of the chunk's tiles
  char* bops;           // [U][ntile_max][NB][2 dhb] B operands
  float* zk;            // saved LayerNorm rows (nullable together)
  float* rk;
  float* zq;
  float* rq;
  long U, P, copy;      // copy: bytes of one operand copy of a unit
  long wunit;           // bytes between units in wops
  long toff;            // bytes from a unit's R high to its T copy
  long wslot, mslot;    // bytes of one slot
  int T, C, NC, dh, ntile_max;
  int keep;             // 1: one slot per chunk (saving), 0: one slot
  int resln;
  float eps;
  const float* ln_a;
  const float* ln_b;
  int H;
  // set per launch
  int r, slot, slot_next, ntile, init, last, items;
};

struct TileBwdArgs {
  const void* q;
  const void* k;
  const void* v;
  const void* d_out;
  const float* kw;
  const float* km;
  const float* carry;
  const char* wops;     // the forward's copies, one slot per chunk
  const char* mops;
  const float* zk;
  const float* rk;
  const float* zq;
  const float* rq;
  const float* d_w_out; // nullable
  const float* d_m_out; // nullable
  float* state;         // [U][Wb | Mb] running adjoint state, fp32 in register-tile order
  float* d_w_in;
  float* d_m_in;
  void* dq;
  void* dk;
  void* dv;
  float* kwb;           // [U][T] adjoints of the scalar kernels
  float* kmb;
  float* carryb;        // [slots][U][NC][3], one slot per state workgroup of a unit
  char* gops;           // [U][R of Wb | T of Wb | R of Mb | T of Mb]
  char* aops;           // key side: [U][ntile_max][dY, Yh, K], [A, dAh, Hh..]
  char* bops;
  char* qaops;          // query side: [U][ntile_max][Yb_Q, Q], [A_Q, Hb_Q..] (ahead of a
  char* qbops;          // chain [U][NC][ntile_max])
  float* ln_zbar;       // with the affine: adjoint of a e
  long U, P, copy, wunit, wslot, mslot;
  int T, C, NC, dh, ntile_max;
  int resln;
  const float* ln_a;
  const float* ln_b;
  int H;
  int r, ntile, init, last;
};

// Whether the path has kernels for a net and its shape.
bool tile_supported(const ChainConfig& cfg, int dh);
// Bytes of one tile's A and B operands: of the forward, of the backward's key
// side, of its query side.
enum TileOps { kTileFwd, kTileBwdKey, kTileBwdQuery };
long tile_aop_bytes(const ChainConfig& cfg, TileOps ops);
long tile_bop_bytes(const ChainConfig& cfg, int dh, TileOps ops);
// State workgroups of a unit: the slots of carryb.
int tile_state_groups(int dh);
hipError_t launch_tile_fwd(const ChainConfig& cfg, const TileFwdArgs& a, hipStream_t s);
hipError_t launch_tile_bwd(const ChainConfig& cfg, const TileBwdArgs& a, hipStream_t s);
// The query sides alone, for a chain that leaves them out: the forward's of
// chunks [a.r, a.r + nchunks), the backward's of all chunks (ntile_max tiles each).
hipError_t launch_tile_fwd_query(const ChainConfig& cfg, TileFwdArgs a, int nchunks, hipStream_t s);
hipError_t launch_tile_bwd_query(const ChainConfig& cfg, const TileBwdArgs& a, hipStream_t s);

}  // namespace e2ttt

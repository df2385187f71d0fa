// carve_kernels.h -- kernel argument blocks, LDS layouts and launch entry
// points shared by the CARVE HIP translation units.
#pragma once
#include "../../include/carve.h"
#include "carve_dev.h"

namespace carve {

// Kernel variants (template argument VAR, a bit set):
//   kVarGated:   the decay g is formed in the kernels from its raw logit f
//                (Eq. decay_gate: g = -exp(A) softplus(f + tau_f));
//   kVarScalarW: the scalar write gate (Sec. scalar write gate): one logit wx
//                per (token, head), w = sigmoid(wx) on every value channel and
//                no content term on the write side, so the fold is F = Ub S_hat
//                (R rows instead of 2R) and there is no Uw, Vw;
//   kVarAct:     q, k, v are the raw projections; the kernels apply the input
//                activations (Sec. input projections, Fig. carve_block): q, k =
//                SiLU then L2 normalisation over d_k, v = SiLU.
// Built: every combination of kVarGated and kVarScalarW, and kVarAct alone.
enum : int { kVarGated = 1, kVarScalarW = 2, kVarAct = 4 };
__host__ __device__ constexpr bool var_built(int var) { return var >= 0 && var <= kVarAct; }

// rows of the fold F (and columns of tau) of a variant, R padded to RP:
// [Ub; 0; Uw; 0], or [Ub; 0] with the scalar write gate
__host__ __device__ constexpr int fold_rows(int RP, int var) { return (var & kVarScalarW) ? RP : 2 * RP; }

// ---- forward ----------------------------------------------------------------
struct FwdArgs {
  const void *q, *k, *v, *beta, *bx, *wx;   // token tensors (dtype of the call);
                                            // wx is [B,T,H] with the scalar write gate
  const float *g, *Ub, *Uw, *Vb, *Vw, *S0;  // f32 (Uw, Vw unused with the scalar write gate)
  // decay gate from its raw logit (gated kernels; Eq. decay_gate): f [B,T,H,Dk]
  // in the token dtype, A and tau_f [H,Dk] f32; g is unused then
  const void* f;
  const float *A, *tau_f;
  void* o;
  float *S_T, *S_chunks;
  void* rec;     // chunk records (recompute mode of the backward)
  int B, T, H, R, RP, L;
};

// ---- rows of D token-dtype elements as matrix-core operands ---------------------
// Row stride (elements) and element-index XOR of a [rows][D] operand tile whose
// quads (4 elements, 8 bytes in bf16) are read along a row (in pairs 16 columns
// apart, one LDS instruction) and across rows and written as result quads: bf16
// rows of 16 (mod 32) elements with qswz, f32 rows with a 16-byte pad.
template <typename T, int D>
struct RowTile {
  static constexpr int LD = sizeof(T) == 2 ? (D % 32 == 16 ? D : D + 16) : D + 4;
  static __device__ __forceinline__ int sw(int r) { return qswz<T>(r); }
  // element offset of (row r, column c0 + q), c0 a multiple of 16 and q = 0, 4, 8
  // or 12 (the swizzle moves q only, so offsets along a row stay immediate)
  static __device__ __forceinline__ int at(int r, int c0, int q) { return r * LD + c0 + (q ^ sw(r)); }
  // lane (g, c) receives tile[r0 + 4 g + e][c0 + c], e = 0..3 (r0, c0 multiples of 16)
  static __device__ __forceinline__ typename Quad<T>::q tr(const T* t, int r0, int c0, int g, int c) {
    return Quad<T>::ld_tr_sw(t, LD, r0, c0, g, c);
  }
};
// The layer's parameters as matrix-core operands.  A workgroup takes them once,
// at its start, where nothing hides a load: every load is issued before the
// first use (rows and columns past R read a valid address and are zeroed by a
// select, not skipped by a branch), so that they cost one memory latency
// together with the first block's own loads (one 16-token chunk of 256 chains at
// d = 128: 20.2 us with element loads one after another, 16.5 us now).
// [Ub; 0; Uw; 0] (or [Ub; 0] with the scalar write gate) in the token dtype as a
// RowTile; 4 D threads, 16 rows of 16-byte loads at a time
template <typename T, int D, int RP, bool SW>
__device__ __forceinline__ void stage_U(T* sU, const float* Ub, const float* Uw, int R, int tid) {
  constexpr int N = (SW ? RP : 2 * RP) / 16;
  const int r0 = tid / (D / 4), i = 4 * (tid % (D / 4));
  f32x4 v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int r = 16 * (u % (RP / 16)) + r0;
    v[u] = gload4((u < RP / 16 ? Ub : Uw) + (r < R ? r : 0) * D + i);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int r = 16 * (u % (RP / 16)) + r0;
    Quad<T>::st(sU + RowTile<T, D>::at(16 * u + r0, i & ~15, i & 12), Quad<T>::cvt(r < R ? v[u] : zero4()));
  }
}
// operand quads of row `row` of V [rows][R], lane group g: V[row][16 ks + 4 g + e]
template <typename T, int RP>
__device__ __forceinline__ void load_V(typename Quad<T>::q (&f)[RP / 16], const float* V, int R, int row, int g) {
  f32x4 t[RP / 16];
#pragma unroll
  for (int ks = 0; ks < RP / 16; ++ks)
    for (int e = 0; e < 4; ++e) {
      const int r = 16 * ks + 4 * g + e;
      t[ks][e] = V[row * R + (r < R ? r : 0)];
    }
#pragma unroll
  for (int ks = 0; ks < RP / 16; ++ks) {
    for (int e = 0; e < 4; ++e) t[ks][e] = 16 * ks + 4 * g + e < R ? t[ks][e] : 0.0f;
    f[ks] = Quad<T>::cvt(t[ks]);
  }
}
// 16 x 16 coupling tiles (A, P, T, dA, dP), one after another: rows of 16
// elements with qswz (bf16), or 20 (f32)
template <typename T>
struct SmallTile {
  static constexpr int LD = sizeof(T) == 2 ? 16 : 20;
  static constexpr int N = 16 * LD;   // elements of a tile
  static __device__ __forceinline__ int at(int r, int col) { return r * LD + (col ^ qswz<T>(r)); }
  static __device__ __forceinline__ typename Quad<T>::q tr(const T* t, int g, int c) {
    return Quad<T>::ld_tr_sw(t, LD, 0, 0, g, c);
  }
  // T x (or T^T x) for a unit triangular T, from its tile's operand quads: bf16
  // tiles hold T - I and x enters once more in f32, so that its rounding to an
  // operand meets T - I only (2-norm errors against 64 bits, layer with B = 4,
  // H = 16, T = 4096, d = 128: dv 3.74e-3 with T itself, 3.34e-3 now, dk 3.74e-3
  // and 3.37e-3, dg 3.74e-3 and 3.40e-3); f32 tiles hold T
  static __device__ __forceinline__ f32x4 apply_T(typename Quad<T>::q t, f32x4 x) {
    return Quad<T>::mma16(t, Quad<T>::cvt(x), sizeof(T) == 2 ? x : f32x4{0.0f, 0.0f, 0.0f, 0.0f});
  }
};

// Lower-triangular 16-token tile pairs (i, j) of a block of NB tiles, row-major:
// inclusive (j <= i) and strict (j < i) enumeration.
__host__ __device__ constexpr int tri_incl(int i, int j) { return i * (i + 1) / 2 + j; }
__host__ __device__ constexpr int tri_strict(int i, int j) { return i * (i - 1) / 2 + j; }
// coupling tiles of a block: P (inclusive), -A (strict), T (one per tile)
__host__ __device__ constexpr int tiles_p(int NB) { return NB * (NB + 1) / 2; }
__host__ __device__ constexpr int tiles_a(int NB) { return NB * (NB - 1) / 2; }
__host__ __device__ constexpr int tiles_all(int NB) { return tiles_p(NB) + tiles_a(NB) + NB; }

// Per-(batch, head, chunk) record written by the chunk-parallel recompute of
// the backward and read by its adjoint (byte offsets, 256-aligned).  The chunk
// is L / (16 NB) WY blocks of NB 16-token tiles; NT threads per workgroup, RF
// fold rows (fold_rows), thread tid = 64 w + 16 g + c.  "Thread order": the
// 4-element vector of thread tid at index tid, so that a wave reads and writes
// it in whole lines; "tile image": the bytes of the adjoint's LDS tile.
//   FT   [RF/16][NT] quads      F[16 rt + 4 g + e][16 w + c]
//   Tau  [L][RF]                tanh(q F^T), plain rows
//   K    per block [3][16 NB] rows, tile images: beta Kt, Qt, Ki
//   U    per block [16 NB] rows, tile image: u
//   C    per block tiles_all(NB) coupling tiles, tile images: P, -A, T (bf16: T - I)
//   S    [L/16][D/16][NT] quads S'[16 vt + 4 g + e][16 w + c], the block start
//                               state times the block's reference e^{rho}: entry
//                               NB m of block m, or (per-tile evaluation) entry
//                               NB m + i of its tile i
//   Gam  [L/16][D] f32          e^{rho}, indexed like S
//   Beta [2][L] f32             beta, then the scalar write gate sigmoid(wx)
//   E    [L/16][NT] f32x4       e^{lam_t - rho}: t = 16 tt + c, keys 16 w + 4 g + e
//   Sig  [L/16][NT] quads       the erase gate, same elements
//   W    [L/16][NT] f32x4       the write gate: t = 16 tt + 4 g + e, value 16 w + c
//                               (not with the scalar write gate)
//   V    [L/16][NT] quads       v (activated), same elements
//   Q    [L/16][NT] quads       q (activated): t = 16 tt + 4 g + e, key 16 w + c
//   dF   [D][RF] f32            written by the adjoint: the chunk's gradient of F,
//                               stored transposed (dF[r][j] at (j, r))
struct ChunkRec {
  unsigned FT, Tau, K, U, C, S, Gam, Beta, E, Sig, W, V, Q, dF;
  unsigned total;
};
__host__ __device__ constexpr unsigned rec_align(unsigned x) { return (x + 255) & ~255u; }
// bytes of one [rows][D] tile image and of one block's coupling tiles
template <typename T, int D>
__host__ __device__ constexpr unsigned image_bytes(int rows) { return (unsigned)(rows * RowTile<T, D>::LD * (int)sizeof(T)); }
template <typename T>
__host__ __device__ constexpr unsigned ctile_bytes(int NB) { return (unsigned)(tiles_all(NB) * SmallTile<T>::N * (int)sizeof(T)); }

template <typename T, int D>
__host__ __device__ constexpr ChunkRec chunk_rec(int L, int RF, int NB) {
  ChunkRec r{};
  const unsigned e = sizeof(T), nt = L / 16, NT = (D / 16) * 64;
  unsigned off = 0;
  r.FT = off;  off += rec_align((RF / 16) * NT * 4 * e);
  r.Tau = off; off += rec_align(L * RF * e);
  r.K = off;   off += rec_align(3 * image_bytes<T, D>(L));
  r.U = off;   off += rec_align(image_bytes<T, D>(L));
  r.C = off;   off += rec_align((nt / NB) * ctile_bytes<T>(NB));
  r.S = off;   off += rec_align(nt * D * D * e);
  r.Gam = off; off += rec_align(nt * D * 4);
  r.Beta = off; off += rec_align(2 * L * 4);
  r.E = off;   off += rec_align(nt * NT * 16);
  r.Sig = off; off += rec_align(nt * NT * 4 * e);
  r.W = off;   off += rec_align(nt * NT * 16);
  r.V = off;   off += rec_align(nt * NT * 4 * e);
  r.Q = off;   off += rec_align(nt * NT * 4 * e);
  r.dF = off;  off += rec_align(RF * D * 4);
  r.total = off;
  return r;
}

// threads of a forward workgroup: one wave per 16-wide tile of the key (and
// value) axis
__host__ __device__ constexpr int fwd_threads(int D) { return (D / 16) * 64; }
// threads of a backward workgroup: one wave per 16-column tile of the state
__host__ __device__ constexpr int bwd_threads(int D) { return (D / 16) * 64; }

// LDS per workgroup on gfx950
constexpr size_t kMaxLdsBytes = 160 * 1024;

__host__ __device__ constexpr size_t lds_round(size_t x) { return (x + 15) & ~(size_t)15; }
__host__ __device__ constexpr size_t lds_max(size_t a, size_t b) { return a > b ? a : b; }

// LDS layout of the chunk recompute for WY blocks of NB 16-token tiles (W = 16 NB
// tokens).  X holds the chunk start state while the fold reads it, then the
// block's rows of v and wx until the gates have taken them, then S diag(e^{rho})
// for its transposition; Kt holds the erase logits, Qt the queries and Ki the
// keys until the gates replace them with the decayed operands in place.  Beta
// holds beta, then the scalar write gates.
struct RecLds {
  size_t U, X, Kt, Qt, Ki, F, Tau, C, Gam, Flag, Beta, total;
};

template <typename T, int D, int RP, int VAR, int NB>
__host__ __device__ constexpr RecLds rec_lds() {
  RecLds l{};
  const size_t e = sizeof(T);
  constexpr size_t RF = fold_rows(RP, VAR), W = 16 * NB;
  constexpr size_t im = lds_round(image_bytes<T, D>(W));
  size_t off = 0;
  l.U = off;    off += lds_round(RF * RowTile<T, D>::LD * e);
  l.X = off;    off += lds_max(lds_round(image_bytes<T, D>(D)), 2 * im);
  l.Kt = off;   off += im;
  l.Qt = off;   off += im;
  l.Ki = off;   off += im;
  l.F = off;    off += lds_round(RF * RowTile<T, D>::LD * e);
  l.Tau = off;  off += lds_round(W * RowTile<T, (int)RF>::LD * e);
  l.C = off;    off += lds_round(ctile_bytes<T>(NB));
  l.Gam = off;  off += lds_round((size_t)NB * D * 4);
  l.Flag = off; off += lds_round(16 * 4);
  l.Beta = off; off += lds_round(2 * W * 4);
  l.total = off;
  return l;
}

// LDS layout of the chain forward for one WY block of WB tokens (NB = WB / 16
// token tiles); SW: the scalar write gate (RP fold rows instead of 2RP).  Rows
// of n columns take fwd_qstride(n) elements (bf16: 16 (mod 32), the quad
// swizzle qswz; f32: a 16-byte pad).  Region X holds the chunk start
// state while the fold reads it, then the block's raw erase logits (Bx) and the
// decayed keys Kt; Ki holds the block's raw keys until the gates turn them
// into Ki in place.
// With VW (when the layout still fits), VW holds the block's value-side token
// tiles (v, wx: WB rows each, unpadded, 16-byte chunks XOR-swizzled by row) from
// the first barrier of a block to its gates; it overlays A .. TmT, which are
// written only after the gates.  Without VW those tiles are read per wave.
// Tab holds the block's per-channel factor tables, Flag one word per wave
// (whether one of its key channels needs per-tile references).
// Beta holds beta and (scalar write gate) w of the block, for two blocks.
struct ChainLds {
  size_t U, X, Kt, Bx, Ki, F, Q, Tau, A, P, TmT, VW, Tab, Flag, Beta, Gate, total;
};

// Per-channel factor tables of a forward WY block of NB 16-token tiles
// (carve_fwd_chain.h), m_i the reference of tile i and c_i the log retention
// at its end: e^{m_i} (NB rows), e^{lam_end - m_i} (NB), e^{c_i - m_i} (NB),
// e^{lam_end} (1) and e^{m_i - c_j} for i >= j + 2 ((NB - 1) (NB - 2) / 2).  A
// block of one tile needs only e^{m_0}.
// A forward block takes one reference per key channel while every channel's
// log retention over the block stays above -kWideLog (factors up to
// e^{kWideLog / 2}), per-tile references otherwise.
constexpr float kWideLog = 160.0f;
// The backward's bound is half of that (factors up to e^{kBwdWideLog / 2} =
// 2e17): its state gradient and block start state meet these factors as bf16
// operands, e^{rho} dS among them, and gradients are often small.  With 160,
// gradients of 1e-6 lost their part through a channel that decays by 2.4 per
// token (e^{-77} 1e-6 is below bf16's range): dk was wrong by 6.7 % (2-norm; with
// blocks of 16 tokens 0.4 %).  Layers whose channels decay by up to one per
// token stay on the one-reference evaluation.
constexpr float kBwdWideLog = 80.0f;
__host__ __device__ constexpr int fwd_tab_rows(int NB) {
  return NB == 1 ? 1 : 3 * NB + 1 + (NB - 1) * (NB - 2) / 2;
}

// Row stride (elements) of a forward operand tile with n columns: bf16 tiles
// take the quad swizzle qswz and need a stride of 16 (mod 32) elements (4 (mod
// 8) quads); f32 tiles keep a 16-byte pad.
template <typename T>
__host__ __device__ constexpr int fwd_qstride(int n) {
  return sizeof(T) == 2 ? (n % 32 == 16 ? n : n + 16) : n + 16 / (int)sizeof(T);
}

template <typename T, int D, int WB, int RP, int VAR, bool VW>
__host__ __device__ constexpr ChainLds chain_lds_v() {
  ChainLds l{};
  const size_t e = sizeof(T);
  constexpr bool SW = (VAR & kVarScalarW) != 0;
  constexpr size_t RF = fold_rows(RP, VAR);
  constexpr size_t NB = WB / 16;
  constexpr size_t LDD = fwd_qstride<T>(D), LDR = fwd_qstride<T>(RF), LDW = fwd_qstride<T>(WB),
                   LDB = fwd_qstride<T>(16);
  size_t off = 0;
  l.U = off;    off += lds_round(RF * LDD * e);
  l.X = off;    off += lds_round(lds_max(D * LDD * e, 2 * lds_round(WB * LDD * e)));
  l.Kt = l.X;
  l.Bx = l.X + lds_round(WB * LDD * e);
  l.Ki = off;   off += lds_round(WB * LDD * e);
  l.F = off;    off += lds_round(RF * LDD * e);
  l.Q = off;    off += lds_round(WB * LDD * e);
  l.Tau = off;  off += lds_round(WB * LDR * e);
  l.A = off;    off += lds_round(WB * LDW * e);
  l.P = off;    off += lds_round(WB * LDW * e);
  l.TmT = off;  off += lds_round(NB * 16 * LDB * e);
  l.VW = l.A;
  if (VW) off = lds_max(off, l.VW + lds_round(2 * WB * (size_t)D * e));
  l.Tab = off;  off += lds_round((size_t)fwd_tab_rows((int)NB) * D * 4);
  l.Flag = off; off += lds_round(16 * 4);   // one word per wave
  l.Beta = off; off += lds_round((SW ? 4 : 2) * WB * 4);
  l.Gate = off; off += lds_round(2 * D * 4);   // -exp(A), tau_f of the head (gated)
  l.total = off;
  return l;
}

// whether the value-side tiles are staged (the layout with VW fits)
template <typename T, int D, int WB, int RP, int VAR>
__host__ __device__ constexpr bool chain_stage_vw() {
  return chain_lds_v<T, D, WB, RP, VAR, true>().total <= kMaxLdsBytes;
}

template <typename T, int D, int WB, int RP, int VAR>
__host__ __device__ constexpr ChainLds chain_lds() {
  return chain_lds_v<T, D, WB, RP, VAR, chain_stage_vw<T, D, WB, RP, VAR>()>();
}

// forward of the whole sequence (one workgroup per (batch, head)), WY blocks of
// WB tokens; launch_chain_fwd dispatches on var to launch_chain_fwd_var<VAR>
// (each variant is compiled in a translation unit of its own)
int launch_chain_fwd(const FwdArgs& a, int dtype, int D, int WB, int var, hipStream_t s);
template <int VAR>
int launch_chain_fwd_var(const FwdArgs& a, int dtype, int D, int WB, hipStream_t s);
// LDS bytes of the chain forward of the default variant (2RP fold rows)
size_t chain_lds_bytes(int dtype, int D, int WB, int RP);


// ---- backward -----------------------------------------------------------------
struct BwdArgs {
  const void* v;    // the raw values (activated inputs); the rest comes from the records
  const float *Ub, *Uw, *Vb, *Vw;
  const float* S_chunks;
  const void* dO;
  const float* dS_T;
  void *dq, *dk, *dv, *dbeta, *dbx, *dwx;   // dwx [B,T,H] with the scalar write gate
  float* dg;
  // gated kernels: decay logit and its parameters, df (token dtype) instead of
  // dg, per-(b,h) partial dA, dtau ([B*H][2][Dk] f32, workspace)
  const void* f;
  const float *A, *tau_f;
  void* df;
  float* partG;
  float* dS0;
  float* part;    // per-(b,h, chunk split) partial d[Ub; Uw] (workspace)
  float* partV;   // per-(b,h,split) partial dVb, dVw (workspace)
  const void* rec;  // chunk records of the recompute (workspace)
  void* opnd;       // per-(b,h) operand quads of the parameters (workspace, adj_opnd_bytes each)
  int B, T, H, R, RP, L, NB;   // NB: 16-token tiles of a WY block of the backward
  int splits;       // chunk and token splits of the parameter gradients per (batch, head)
  int wait_limit;   // polls of the adjoint's bounded wait for a chunk record
};

// Splits per (batch, head) of the parameter-gradient partials: chunk splits of
// d[Ub; Uw], token splits of dVb, dVw.  Each kind gets at least kParamItems
// workgroups (two per compute unit, which keep the reads in flight since each
// loads a step ahead); more splits than that only add partial records to write
// and to sum: with 16 always, a training step at B*H = 128, T = 2048, d = 128
// took 1337 us and now takes 1314; at B*H = 64, T = 4096 2182 and 2174 (up to
// B*H = 32 nothing changes).
constexpr int kMaxParamSplits = 16;
constexpr int kParamItems = 512;
__host__ __device__ constexpr int param_splits(int nbh) {
  return nbh * kMaxParamSplits <= kParamItems ? kMaxParamSplits : (kParamItems + nbh - 1) / nbh;
}

// LDS layout of the adjoint for WY blocks of NB 16-token tiles (W = 16 NB
// tokens).  dM holds the state gradient for the key side, then (from the
// pair-term step on) the write-logit gradients dz_w and, behind them, dY; R the
// exchanged -dR, then dz_b; C the block's coupling tiles, then dA and dP; U and
// dO at a chunk start the two token-dtype parts of dF.  Dbeta and Dwx hold one
// row of partial sums per wave.
struct AdjLds {
  size_t Kt, Qt, Ki, U, dO, dM, R, C, dY, Dbeta, Dwx, Beta, Ws, Gam, Ctl, total;
};

template <typename T, int D, int RP, int VAR, int NB>
__host__ __device__ constexpr AdjLds adj_lds() {
  AdjLds l{};
  const size_t e = sizeof(T);
  constexpr bool SW = (VAR & kVarScalarW) != 0;
  constexpr size_t RF = fold_rows(RP, VAR), W = 16 * NB, NW = D / 16;
  constexpr size_t im = lds_round(image_bytes<T, D>(W));
  size_t off = 0;
  l.Kt = off;    off += im;
  l.Qt = off;    off += im;
  l.Ki = off;    off += im;
  l.U = off;     off += im;
  l.dO = off;    off += im;
  // dF parts over U and dO: bf16 two unpadded [D][RF] tiles, f32 one padded
  constexpr size_t df = sizeof(T) == 2 ? 2 * D * RF * 2 : (size_t)D * (RF + 4) * 4;
  off = lds_max(off, l.U + lds_round(df));
  l.dM = off;
  l.dY = l.dM + (SW ? 0 : im);
  off += lds_max(lds_round(image_bytes<T, D>(D)), (SW ? 0 : im) + lds_round(W * RowTile<T, (int)RF>::LD * e));
  l.R = off;     off += im;
  l.C = off;     off += lds_round(lds_max(ctile_bytes<T>(NB), (size_t)2 * tiles_p(NB) * SmallTile<T>::N * e));
  l.Dbeta = off; off += lds_round(NW * W * 4);
  l.Dwx = off;   off += SW ? lds_round(NW * W * 4) : 0;
  l.Beta = off;  off += lds_round(W * 4);
  l.Ws = off;    off += SW ? lds_round(W * 4) : 0;
  l.Gam = off;   off += lds_round(D * 4);
  l.Ctl = off;   off += 16;
  l.total = off;
  return l;
}

// LDS of the fused chunk recompute + adjoint launch
template <typename T, int D, int RP, int VAR, int NB>
__host__ __device__ constexpr size_t fused_lds() {
  return lds_max(rec_lds<T, D, RP, VAR, NB>().total, adj_lds<T, D, RP, VAR, NB>().total);
}

// bytes of one adjoint workgroup's parameter operands: V^T of the dtau tiles (RF
// x D spread over the waves, at least one fold row tile each) and [Ub; Uw] (RF
// x D) as token-dtype quads, then -exp(A) and tau_f (gated) as f32 vectors, all
// in thread order
__host__ __device__ constexpr size_t adj_opnd_quads(int D, int RF) {
  const size_t nw = D / 16, nrt = RF / 16, nvs = nrt < nw ? 1 : nrt / nw;
  return (nvs * nw + nrt) * nw * 64;
}
__host__ __device__ constexpr size_t adj_opnd_bytes(int D, int RF, size_t e) {
  return adj_opnd_quads(D, RF) * 4 * e + 2 * (size_t)(D / 16) * 64 * 16;
}

// Chunk recompute and adjoint in one launch (see carve_bwd.h).  f carries the
// forward inputs, S_chunks and the chunk records (f.rec == a.rec); sync points
// at sync_ints(B * H, T / L) ints of workspace, zeroed by launch_sync_clear
// on the same stream before; cus is the device's compute-unit count.
// launch_bwd_fused dispatches on var to launch_bwd_fused_var<VAR>.
int launch_bwd_fused(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, int dtype, int D, int NB,
                     int var, hipStream_t s);
template <int VAR>
int launch_bwd_fused_var(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, int dtype, int D, int NB,
                         hipStream_t s);
// dA[h][j], dtau[h][j] = sums over b (in order) of the per-(b,h) partials
int launch_gate_reduce(const float* partG, int B, int H, int D, float* dA, float* dtau, hipStream_t s);
int launch_sync_clear(int* sync, size_t n, hipStream_t s);
// LDS bytes of the fused launch with WY blocks of NB 16-token tiles (the
// largest over the variants), and bytes of one chunk record
size_t bwd_lds_bytes(int dtype, int D, int NB, int RP);
size_t chunk_rec_bytes(int dtype, int D, int L, int RF, int NB);
// ints of the synchronisation area: one ready flag per chunk, the ticket
// counter that assigns the workgroup roles, the wait-timeout word (nonzero once
// an adjoint wave's bounded wait for a record ran out), padding, then per
// (batch, head) the adjoint's position, which paces the recompute: 0 before it
// runs, then 1 + the chunks it has started (counted from the last)
__host__ __device__ constexpr size_t sync_ints(size_t nbh, size_t nch) { return nbh * nch + 4 + nbh; }
__host__ __device__ constexpr size_t sync_ticket(size_t nbh, size_t nch) { return nbh * nch; }
__host__ __device__ constexpr size_t sync_timeout_word(size_t nbh, size_t nch) { return nbh * nch + 1; }
__host__ __device__ constexpr size_t sync_adjoint_pos(size_t nbh, size_t nch) { return nbh * nch + 4; }
// Bound of the adjoint's wait for a chunk's flag: 2^20 polls (each a device-scope
// load and a short sleep; about a second in all).  A chunk is recomputed in tens
// of microseconds, by a workgroup that waits for at most kLeadSpinLimit polls of
// its own once, so the bound is not reached in a correct launch; if it is, every
// wave poisons its state gradient with NaN (every gradient of earlier tokens
// then comes out NaN), the wait-timeout word is set and the workgroup waits no
// more.  It is a kernel argument (BwdArgs::wait_limit, this unless a test sets
// it) so that tests can make the wait give up from the host while every kernel
// still runs to completion.
constexpr int kReadySpinLimit = 1 << 20;
// d[Ub; Uw] over chunk splits and dVb, dVw over token splits (carve_param.h),
// one launch; sw: the scalar write gate (dVb, dUb only; the records hold RP
// fold rows)
int launch_bwd_param(const BwdArgs& a, int dtype, int D, bool sw, hipStream_t s);
// in one launch: sum npartU records of 2 * half floats at partU into dU0 (first
// half) and dU1, and npartV records at partV into dV0 and dV1; with dU1 == dV1
// == NULL only the first halves are summed
int launch_param_reduce(const float* partU, int npartU, const float* partV, int npartV, size_t half, float* dU0,
                        float* dU1, float* dV0, float* dV1, hipStream_t s);
// kVarAct: turn dq, dk (gradients of the activated q, k, in place, [rows][D]) into
// the gradients of the raw projections q_raw, k_raw
int launch_act_bwd(const void* q_raw, const void* k_raw, void* dq, void* dk, size_t rows, int D, int dtype,
                   hipStream_t s);

// Output RMS normalisation over rows of N = H * Dv values (carve_norm.hip).
// The backward's workgroups (at most kNormBwdGroups) each write one f32
// partial row of dweight, summed in order by a second launch; mark (if not
// NULL) is called between the two launches.
constexpr int kNormBwdGroups = 1024;
// carve_rmsnorm_bwd_noalloc: bytes of the per-device static scratch (every
// supported row length: kNormBwdGroups partial rows of up to 4096 floats) and
// the devices it can address
constexpr size_t kNormScratchBytes = (size_t)kNormBwdGroups * 4096 * sizeof(float);
constexpr int kMaxNormDevices = 64;
int norm_scratch(float** ptr);
bool rmsnorm_supported(int dtype, int N);
int rmsnorm_bwd_groups(long rows);
int launch_rmsnorm_fwd(const void* x, const float* wt, void* y, long rows, int N, float eps, int dtype,
                       hipStream_t s);
int launch_rmsnorm_bwd(const void* x, const float* wt, const void* dy, void* dx, float* partial, float* dw, long rows,
                       int N, float eps, int dtype, hipStream_t s, void (*mark)(hipStream_t));

// floats of one partial-gradient record: d[Ub; Uw] ([R][D] twice) or dVb, dVw ([D][R] twice)
__host__ __device__ constexpr size_t part_floats(int R, int D) { return (size_t)2 * R * D; }

}  // namespace carve

// carve_bwd.h -- chunked CARVE backward on gfx950 (App. Alg. backward): the
// chunk recompute + adjoint kernel templates (instantiated per variant in
// carve_variant.hip; the other launches are in carve_bwd.hip).
//
// The backward runs as a sequence of launches on one stream:
//   1. carve_sync_clear_kernel: zeroes the chunk ready flags and the ticket
//      counter of step 2 (a fill kernel, so the sequence may be graph-captured);
//   2. carve_bwd_fused_kernel: two kinds of workgroup in one grid.
//      Recompute workgroups (rec_run, carve_rec.h) recompute chunks
//      independently from S_chunks, latest chunks first, and write a chunk
//      record each, then raise that chunk's ready flag.  Adjoint workgroups
//      (Adjoint below), one per (batch, head), walk the chunks and their WY
//      blocks in reverse, carry the state gradient and wait for a chunk's flag
//      before reading its record, so the recompute runs on the compute units
//      the adjoint leaves idle, ahead of it;
//   3. carve_bwd_param_kernel: d[Ub; Uw] from the per-chunk dF (parked in the
//      chunk records by step 2) and the chunk start states, split over
//      chunks, and dVb, dVw from dbx, dwx and tau, split over tokens;
//   4. carve_param_reduce_kernel: fixed-order sums of the parameter partials,
//      so reruns are bitwise identical.
//
// Adjoint of one WY block of NB 16-token tiles (wave w owns value tile w and
// key tile w; the state gradient dS lives in registers as dS^T tiles, rows = key
// index j, columns = the wave's 16 value rows).  The block is evaluated
// relative to the per-key-channel reference rho = lam_end / 2, the middle of
// its log-retention range.  With S' = S diag(e^{rho}) the scaled block start
// state, gam = e^{rho}, dS_end the gradient of the block end state (S' + u^T Ki)
// diag(gam), and lam, Kh = beta Kt, Qt, Ki (relative to rho), A, P, T, R, u as in
// the recompute:
//   dM   = dS_end diag(gam)
//   du   = Ki dM^T + P^T dO             (du_s = dM Ki_s + sum_t P_ts dO_t)
//   dR   = (I + A)^{-T} du              (blocked back substitution with T_ii, A_ij)
//   dS   = (dM + dO^T Qt - dR^T Kh) diag(e^{rho})   (gradient at the block start)
//   y    = -dR S' + dA Ki               dA = -dR u^T (s < t)
//   dQt  = dO S' + dP Ki                dP = dO u^T  (s <= t)
//   dKi  = dM^T u + dA^T Kh + dP^T Qt
//   dKt  = beta y,   d(beta w v) = dR
//   dbeta = rowsum(dR (w v)) + rowsum(Kt y)
//   dgam gam = diag(dM^T S') + sum_s Ki_s (dM^T u_s)
//   dlam_t = dQt_t Qt_t - dKi_t Ki_t + y_{t+1} Kh_{t+1} + [t = end] dgam gam
//   dl = suffix sums of dlam;  dg = dl;  dz_b = -dl b
//   dk = dKt e^{lam_{t-1} - rho} + dKi e^{rho - lam_t},  dq = dQt e^{lam_t - rho} + dY F
// rho is a constant of the block (the block's result does not depend on it), so
// the gradients through lam are those above with rho held fixed.  The factors
// Kh, Qt, Ki that multiply their gradients in dlam and dgam are the token-dtype
// values of the operand tiles, exactly as the products consumed them: the pair
// terms of A and P (and the u^T Ki term of the state carry) enter dlam twice
// with opposite signs and cancel in the suffix sums only then (bf16: with one
// factor unrounded, about 1 % of dl is left instead of 0.2 %).
//   dv = d(wv) w,  dz_w = d(wv) v w (1 - w)
//   dtau = [dz_b Vb, dz_w Vw],  dY = dtau (1 - tau^2),  dF += dY^T q
// and at the chunk start the folded read-out closes the chain ("glue"):
//   dS += [Ub; Uw]^T dF,   d[Ub; Uw] += dF S_hat^T.
// A block that the recompute evaluated tile by tile (carve_rec.h) is walked as
// NB blocks of one tile.  Its images, coupling tiles and dO rows come to LDS with
// those of any other block, loaded while the block before runs, and each tile
// takes its own rows there; what a tile reads from the record beside them is
// loaded during the tile before (at B = 4, H = 16, T = 4096, d = 128 with every
// block of this kind the backward takes 1.92 ms, 2.77 with each tile loaded when
// its turn came; 1.40 with none).
// With the scalar write gate (kVarScalarW; w_t = sigmoid(wx_t) on every value
// channel, no write-side content) the fold is Ub S_hat alone, there is no
// dtau_w, and the gradient of the token's write logit is the sum over the
// value channels: dwx_t = sum_v d(wv)_tv v_tv w_t (1 - w_t).
// With the input activations (kVarAct) the records hold the activated q, k, v,
// and dv is taken through SiLU' here.  dq and dk leave this kernel as gradients
// of the activated q, k; carve_act_bwd_kernel takes them through the L2
// normalisation and SiLU.
#pragma once
#include "carve_rec.h"

namespace carve {

// How many chunks ahead of the adjoint the recompute works: 128 tokens in chunks
// of up to 64, 384 in chunks of 128.  Closer, the adjoint waits for records (one
// chunk of 64 tokens: T = 4096 step 2605 us); further, more records lie in the
// caches between their two uses (2 chunks of 64 tokens 2086 us, 3 2110, 4 2152,
// 6 2223, 8 2226).  16-token chunks take longer per token and want more of them
// (8: 372 us, 4: 389); chunks of 128 tokens are two blocks (1: 1075 us, 2: 1028,
// 3 and 4: 1022).
constexpr int recompute_lead(int L) { return L > 64 ? 3 : 128 / L; }

// Compiler-only fence: keeps the LDS loads of one loop iteration from being
// hoisted above the previous one (bounds the number of live operand registers).
#define CARVE_SEQ() asm volatile("" ::: "memory")

// Adjoint of one (batch, head).  GATED: the kernel writes df = dg (-exp(A))
// sigmoid(f + tau_f) instead of dg and sums dA = dg g and dtau = df over its
// tokens (per lane in registers, reduced once at the end) into a
// per-(batch, head) partial.
//
// The steps of a block are separated by one workgroup barrier each: value side
// (B1), products over the value axis (B2), pair terms and gate gradients (B3),
// dtau (B4), dF / dq and, at a chunk start, the glue (B5).  What a block reads
// from its record reaches the LDS through registers loaded one or two steps
// before their region is free (tile images: linear 16-byte copies), so the
// steps use only LDS, registers and the matrix cores.
template <typename T, int D, int RP, int VAR, int NBK>
struct Adjoint {
  typedef Quad<T> Qd;
  typedef typename Qd::q quad;
  typedef RowTile<T, D> RT;
  typedef SmallTile<T> ST;
  static constexpr bool GATED = (VAR & kVarGated) != 0;
  static constexpr bool SW = (VAR & kVarScalarW) != 0;
  static constexpr bool ACT = (VAR & kVarAct) != 0;
  static constexpr int NT = bwd_threads(D);
  static constexpr int NW = NT / 64;
  static constexpr int NJT = D / 16;
  static constexpr int RF = fold_rows(RP, VAR);
  static constexpr int NRT = RF / 16, NRB = RP / 16;
  typedef RowTile<T, RF> RY;
  static constexpr int VEC = 16 / sizeof(T);
  static constexpr int QB = 4 * (int)sizeof(T);   // bytes of a quad
  static constexpr AdjLds lay = adj_lds<T, D, RP, VAR, NBK>();
  // dtau tiles: wave w takes fold row tiles w % NRW + k NRW (NVS of them) of
  // token tiles w / NRW, + NTW, ...
  static constexpr int NRW = NRT < NW ? NRT : NW;
  static constexpr int NVS = NRT / NRW;
  static constexpr int NTW = NW / NRW;
  static_assert(NRT % NRW == 0 && NW % NRW == 0, "whole tiles per wave");
  // dF parts of the glue: rows of RF elements, quad q of row j at q ^ (j mod 16)
  // (bf16; conflict-free for the row reads and the result-quad writes), or 16
  // bytes of padding (f32, one part)
  static constexpr bool SPLIT = sizeof(T) == 2;
  static constexpr int LDF = SPLIT ? RF : RF + 4;
  static __device__ __forceinline__ int df_at(int j, int r) {
    return j * LDF + (SPLIT ? (r ^ (4 * (j & 15 & (RF / 4 - 1)))) : r);
  }

  const BwdArgs& a;
  const int bh;
  char* smem;
  int tid, lane, w, g, c;
  int H, L, R, nch, mpc, rs, h;
  ChunkRec cr;
  size_t bh0, bh1;
  const char* recb;
  T* opnd;
  // gate constants of the wave's keys (GATED), behind the operand quads
  __device__ __forceinline__ float* gate(int k) const {
    return reinterpret_cast<float*>(opnd + adj_opnd_quads(D, 2 * RP) * 4) + ((size_t)k * NT + tid) * 4;
  }

  // tile images of a block in registers on their way to LDS
  static constexpr int W = 16 * NBK;
  static constexpr int NVK = (int)(image_bytes<T, D>(W) / 16);        // vectors of one image
  static constexpr int NKV = (3 * NVK + NT - 1) / NT, NUV = (NVK + NT - 1) / NT;
  static constexpr int NVC = (int)(ctile_bytes<T>(NBK) / 16);
  static constexpr int NCV = (NVC + NT - 1) / NT;
  static constexpr int NVO = W * D / VEC;                             // vectors of the block's dO rows
  static constexpr int NOV = (NVO + NT - 1) / NT;

  // Opaque copies of the lane coordinates: addresses derived from them are
  // recomputed in every step instead of being kept live across steps and blocks.
  __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(tid), "+v"(g), "+v"(c) : : "memory"); }
  // makes the compiler wait for a loaded value here
  template <typename V>
  static __device__ __forceinline__ void arrived(V& v) { asm volatile("" : "+v"(v)); }
  __device__ __forceinline__ T* lds(size_t off) const { return reinterpret_cast<T*>(smem + off); }
  __device__ __forceinline__ float* ldf(size_t off) const { return reinterpret_cast<float*>(smem + off); }
  __device__ __forceinline__ quad fI() const {
    return Qd::cvt(f32x4{4 * g == c ? 1.0f : 0.0f, 4 * g + 1 == c ? 1.0f : 0.0f, 4 * g + 2 == c ? 1.0f : 0.0f,
                         4 * g + 3 == c ? 1.0f : 0.0f});
  }
  // the transpose of a tile in the result layout, in the token dtype: lane
  // (g, c) receives X[c][4 g + e]
  __device__ __forceinline__ quad tposed(quad x) const { return Qd::cvt(Qd::mma16(x, fI(), zero4())); }

  struct Pre {          // prefetched data of the next block
    u32x4_t k[NKV], cc[NCV], u[NUV], o[NOV];
    f32x4 wg[NBK];
    quad v[NBK];
    f32x4 gam;
    float beta, ws;
  };
  // persistent per-wave values
  struct State {
    f32x4 dS[NJT];      // dS[v = 16 w + c][j = 16 jt + 4 g + i]
    f32x4 gA, gT;       // GATED: sums over this lane's tokens of dg g and df
  };

  // vector u of this thread out of N: threads past the end repeat the last one
  // (the same load and the same LDS write, without a branch around either)
  template <int N>
  __device__ __forceinline__ int vec(int u) const {
    const int x = tid + u * NT;
    return (u + 1) * NT <= N ? x : x < N ? x : N - 1;
  }
  __device__ __forceinline__ const char* rec_of(int ch) const { return recb + (size_t)ch * cr.total; }

  // loads of block (ch, m) into registers
  __device__ __forceinline__ void load_tiles(Pre& p, int ch, int m) const {
    const RecBuf rc(rec_of(ch), cr.total);
    for (int u = 0; u < NKV; ++u) p.k[u] = rc.template ld<u32x4_t>(cr.K + 3 * image_bytes<T, D>(W) * m, 16 * vec<3 * NVK>(u));
    for (int u = 0; u < NCV; ++u) p.cc[u] = rc.template ld<u32x4_t>(cr.C + ctile_bytes<T>(NBK) * m, 16 * vec<NVC>(u));
  }
  __device__ __forceinline__ void load_uo(Pre& p, int ch, int m) const {
    const RecBuf rc(rec_of(ch), cr.total);
    for (int u = 0; u < NUV; ++u) p.u[u] = rc.template ld<u32x4_t>(cr.U + image_bytes<T, D>(W) * m, 16 * vec<NVK>(u));
    const T* so = reinterpret_cast<const T*>(a.dO) + bh0 + (size_t)((ch * L + m * W) * rs);
    for (int u = 0; u < NOV; ++u) {
      const int x = vec<NVO>(u);
      p.o[u] = *reinterpret_cast<const u32x4_t*>(so + (x / (D / VEC)) * rs + (x % (D / VEC)) * VEC);
    }
  }
  __device__ __forceinline__ void load_vals(Pre& p, int ch, int m) const {
    const RecBuf rc(rec_of(ch), cr.total);
    for (int tt = 0; tt < NBK; ++tt) {
      if constexpr (!SW) p.wg[tt] = rc.template ld<f32x4>(cr.W + (m * NBK + tt) * NT * 16, tid * 16);
      p.v[tt] = rc.template ld<quad>(cr.V + (m * NBK + tt) * NT * QB, tid * QB);
    }
  }
  // what one tile of a block evaluated tile by tile takes from the record beside
  // the images
  struct TilePre {
    quad S[NJT], sig, q, v, tau[NVS];
    f32x4 E, wg, gam;
    quad FT[NRT];   // of the chunk
  };
  __device__ __forceinline__ void load_tile(TilePre& t, int ch, int tile) const {
    const RecBuf rc(rec_of(ch), cr.total);
    t.gam = rc.template ld<f32x4>(cr.Gam + tile * D * 4, 16 * vec<D / 4>(0));
    t.v = rc.template ld<quad>(cr.V + tile * NT * QB, tid * QB);
    if constexpr (!SW) t.wg = rc.template ld<f32x4>(cr.W + tile * NT * 16, tid * 16);
    for (int vt = 0; vt < NJT; ++vt) t.S[vt] = rc.template ld<quad>(cr.S + (tile * NJT + vt) * NT * QB, tid * QB);
    t.E = rc.template ld<f32x4>(cr.E + tile * NT * 16, tid * 16);
    t.sig = rc.template ld<quad>(cr.Sig + tile * NT * QB, tid * QB);
    t.q = rc.template ld<quad>(cr.Q + tile * NT * QB, tid * QB);
    for (int k = 0; k < NVS; ++k) t.tau[k] = load_tau(rc, tile, w % NRW + k * NRW);
  }
  __device__ __forceinline__ quad load_tau(const RecBuf& rc, int tile, int rt) const {
    return rc.template ld<quad>(cr.Tau + (16 * tile * RF + 16 * rt) * (int)sizeof(T), (c * RF + 4 * g) * (int)sizeof(T));
  }
  // operands of dF, dq and the glue: [Ub; Uw] and F^T of the chunk
  __device__ __forceinline__ void load_fold(quad (&fU)[NRT], quad (&FT)[NRT], int ch) const {
    const RecBuf rc(rec_of(ch), cr.total);
    for (int rt = 0; rt < NRT; ++rt) fU[rt] = Qd::ld(opnd + ((size_t)(NVS * NJT + rt) * NT + tid) * 4);
    for (int rt = 0; rt < NRT; ++rt) FT[rt] = rc.template ld<quad>(cr.FT + rt * NT * QB, tid * QB);
  }
  // registers -> LDS
  __device__ __forceinline__ void put_gam(f32x4 gam) const {
    *reinterpret_cast<f32x4*>(smem + lay.Gam + 16 * vec<D / 4>(0)) = gam;
  }
  __device__ __forceinline__ void put_tiles(const Pre& p) const {
    u32x4_t* dk = reinterpret_cast<u32x4_t*>(smem + lay.Kt);
    for (int u = 0; u < NKV; ++u) dk[vec<3 * NVK>(u)] = p.k[u];
    u32x4_t* dc = reinterpret_cast<u32x4_t*>(smem + lay.C);
    for (int u = 0; u < NCV; ++u) dc[vec<NVC>(u)] = p.cc[u];
    put_gam(p.gam);
    ldf(lay.Beta)[vec<W>(0)] = p.beta;
    if constexpr (SW) ldf(lay.Ws)[vec<W>(0)] = p.ws;
  }
  // (wide: a block evaluated tile by tile; its last tile's reference comes first)
  __device__ __forceinline__ void load_scalars(Pre& p, int ch, int m, bool wide) const {
    const RecBuf rc(rec_of(ch), cr.total);
    p.gam = rc.template ld<f32x4>(cr.Gam + (m * NBK + (wide ? NBK - 1 : 0)) * D * 4, 16 * vec<D / 4>(0));
    p.beta = rc.template ld<float>(cr.Beta + m * W * 4, 4 * vec<W>(0));
    if constexpr (SW) p.ws = rc.template ld<float>(cr.Beta + (L + m * W) * 4, 4 * vec<W>(0));
  }
  __device__ __forceinline__ void put_uo(const Pre& p) const {
    u32x4_t* du = reinterpret_cast<u32x4_t*>(smem + lay.U);
    for (int u = 0; u < NUV; ++u) du[vec<NVK>(u)] = p.u[u];
    for (int u = 0; u < NOV; ++u) {
      stage_vec<T, D, false, false>(lds(lay.dO), vec<NVO>(u), p.o[u]);
    }
  }

  // Adjoint of one block whose data is in LDS (after a barrier) and p (wg, v; a
  // tile's in tp):
  // tiles tile0 .. tile0 + NB - 1 of chunk ch, which is the whole block in LDS
  // (NB = NBK) or its tile `sub` (NB = 1, a block evaluated tile by tile).
  // NEXT: the next block's data (block next_m of this chunk, or with next_m < 0
  // the last one of chunk wait_ch) is loaded into p meanwhile; otherwise that of
  // the tile before into tp.  wide: the chunk's bits of blocks evaluated tile by tile.
  // wait_ch >= 0: wave 0 waits for that chunk's flag and leaves it in Ctl.
  template <int NB, bool NEXT>
  __device__ __forceinline__ void block(State& s, Pre& p, TilePre& tp, f32x4 (&dF)[NRT], quad (&fU)[NRT], int ch, int tile0, int sub,
                                        int wait_ch, bool& timed_out, int next_m, int wide) {
    constexpr int W = 16 * NB;   // tokens of this block (the images in LDS have 16 NBK rows)
    constexpr int NTP = tiles_p(NB);
    constexpr bool TILE = NB != NBK;
    fresh();
    const RecBuf rc(rec_of(ch), cr.total);
    const int t0 = ch * L + 16 * tile0;
    // a tile takes its own rows of the images, its own coupling tiles (dA over P,
    // dP over T) and the first rows of dM and dY
    const int r0 = TILE ? 16 * sub : 0;
    T* sKt = lds(lay.Kt) + r0 * RT::LD;
    T* sQt = lds(lay.Qt) + r0 * RT::LD;
    T* sKi = lds(lay.Ki) + r0 * RT::LD;
    T* sU = lds(lay.U) + r0 * RT::LD;
    T* sdO = lds(lay.dO) + r0 * RT::LD;
    T* sdM = lds(lay.dM);
    T* sR = lds(lay.R) + r0 * RT::LD;
    T* sP = lds(lay.C) + (TILE ? tri_incl(sub, sub) * ST::N : 0);
    T* sA = lds(lay.C) + tiles_p(NBK) * ST::N;
    T* sT = sA + (tiles_a(NBK) + (TILE ? sub : 0)) * ST::N;
    T* sdA = sP;
    T* sdP = TILE ? sT : lds(lay.C) + NTP * ST::N;
    T* sdY = lds(lay.dY);
    float* sDbeta = ldf(lay.Dbeta) + w * W;
    float* sBeta = ldf(lay.Beta) + r0;
    float* sWs = ldf(lay.Ws) + r0;
    float* sGam = ldf(lay.Gam);
    const auto e0 = [&](int tt) { return (t0 + 16 * tt + c) * rs + 16 * w + 4 * g; };

    // ---- B1: value side (value tile w; rows t = 16 tt + 4 g + i, column v = 16 w + c)
    // S' of the block for B2, loaded ahead of this step's stores (transposed operand quads)
    quad sS[NJT];
    if constexpr (TILE) {
      for (int vt = 0; vt < NJT; ++vt) sS[vt] = tp.S[vt];
    } else {
      for (int vt = 0; vt < NJT; ++vt) sS[vt] = rc.template ld<quad>(cr.S + (tile0 * NJT + vt) * NT * QB, tid * QB);
    }
    quad dOq[NB], nq[NB], dzwT[NB], dvT[NB];   // dO, -dR (K = t operands); dz_w, dv as token rows
    {
      quad dMq[NJT];
      for (int jt = 0; jt < NJT; ++jt) {
        s.dS[jt] *= *reinterpret_cast<const f32x4*>(sGam + 16 * jt + 4 * g);
        dMq[jt] = Qd::cvt(s.dS[jt]);
        Qd::st(sdM + RT::at(16 * w + c, 16 * jt, 4 * g), dMq[jt]);
      }
      for (int tt = 0; tt < NB; ++tt) dOq[tt] = RT::tr(sdO, 16 * tt, 16 * w, g, c);
      f32x4 du[NB];
      for (int tt = 0; tt < NB; ++tt) {
        // (two chains, added at the end: mma16 never accumulates on a mma32 result)
        f32x4 dp = zero4();
        for (int i = tt; i < NB; ++i) dp = Qd::mma16(ST::tr(sP + tri_incl(i, tt) * ST::N, g, c), dOq[i], dp);
        du[tt] = zero4();
        for (int jp = 0; jp < NJT / 2; ++jp)
          du[tt] = Qd::mma32(Qd::ld(sKi + RT::at(16 * tt + c, 32 * jp, 4 * g)), Qd::ld(sKi + RT::at(16 * tt + c, 32 * jp + 16, 4 * g)),
                             dMq[2 * jp], dMq[2 * jp + 1], du[tt]);
        du[tt] += dp;
      }
      f32x4 dR[NB];
      quad xq[NB];
      for (int i = NB - 1; i >= 0; --i) {
        f32x4 r = du[i];
        for (int j = i + 1; j < NB; ++j) r = Qd::mma16(ST::tr(sA + tri_strict(j, i) * ST::N, g, c), xq[j], r);
        dR[i] = ST::apply_T(ST::tr(sT + i * ST::N, g, c), r);
        xq[i] = Qd::cvt(dR[i]);
        nq[i] = Qd::cvt(-dR[i]);
        // exchange: token rows of -dR for the products over the value axis
        Qd::st(sR + RT::at(16 * i + c, 16 * w, 4 * g), tposed(nq[i]));
      }
      // value-side gradients (stored as token rows, 4 values per lane)
      for (int tt = 0; tt < NB; ++tt) {
        const f32x4 bt = *reinterpret_cast<const f32x4*>(sBeta + 16 * tt + 4 * g);
        f32x4 wg;
        if constexpr (SW) wg = *reinterpret_cast<const f32x4*>(sWs + 16 * tt + 4 * g);
        else wg = TILE ? tp.wg : p.wg[tt];
        const f32x4 vv = Qd::f32(TILE ? tp.v : p.v[tt]);
        f32x4 dvv, dzw, pr;
        for (int i = 0; i < 4; ++i) {
          const float dwv = bt[i] * dR[tt][i];
          dvv[i] = dwv * wg[i];
          dzw[i] = dwv * vv[i] * wg[i] * (1.0f - wg[i]);
          pr[i] = row_scan(dR[tt][i] * wg[i] * vv[i]);   // dbeta, value part: sum over v of dR (w v)
        }
        if constexpr (ACT) {
          const f32x4 raw = Qd::f32(Qd::ld(reinterpret_cast<const T*>(a.v) + bh0 + e0(tt)));
          dvT[tt] = Qd::cvt(Qd::mma16(Qd::cvt(dvv), fI(), zero4()) * silu_grad4(raw));
        } else {
          dvT[tt] = tposed(Qd::cvt(dvv));
        }
        if (c == 15) *reinterpret_cast<f32x4*>(sDbeta + 16 * tt + 4 * g) = pr;
        if constexpr (SW) {
          f32x4 pw;
          for (int i = 0; i < 4; ++i) pw[i] = row_scan(dzw[i]);
          if (c == 15) *reinterpret_cast<f32x4*>(ldf(lay.Dwx) + w * W + 16 * tt + 4 * g) = pw;
        } else {
          dzwT[tt] = tposed(Qd::cvt(dzw));
        }
      }
    }
    // the state gradient at the block start
    for (int jt = 0; jt < NJT; ++jt) {
      CARVE_SEQ();
      f32x4 acc = s.dS[jt];
      if constexpr (NB == 1) {
        acc = Qd::mma32(RT::tr(sQt, 0, 16 * jt, g, c), RT::tr(sKt, 0, 16 * jt, g, c), dOq[0], nq[0], acc);
      } else {
        for (int tp = 0; tp < NB / 2; ++tp) {
          acc = Qd::mma32(RT::tr(sQt, 32 * tp, 16 * jt, g, c), RT::tr(sQt, 32 * tp + 16, 16 * jt, g, c), dOq[2 * tp], dOq[2 * tp + 1], acc);
          acc = Qd::mma32(RT::tr(sKt, 32 * tp, 16 * jt, g, c), RT::tr(sKt, 32 * tp + 16, 16 * jt, g, c), nq[2 * tp], nq[2 * tp + 1], acc);
        }
      }
      s.dS[jt] = acc * *reinterpret_cast<const f32x4*>(sGam + 16 * jt + 4 * g);
    }
    __syncthreads();

    // ---- B2: products over the value axis (key tile w; rows j = 16 w + 4 g + i, column t)
    fresh();
    // E and the erase gate for the next step
    f32x4 E[NB];
    quad sig[NB];
    if constexpr (TILE) {
      E[0] = tp.E;
      sig[0] = tp.sig;
    } else for (int tt = 0; tt < NB; ++tt) {
      E[tt] = rc.template ld<f32x4>(cr.E + (tile0 + tt) * NT * 16, tid * 16);
      sig[tt] = rc.template ld<quad>(cr.Sig + (tile0 + tt) * NT * QB, tid * QB);
    }
    // dA = -dR u^T (s < t) and dP = dO u^T (s <= t), stored as rows of t: a wave
    // takes both tiles of a pair (i, j), which share u's rows
#pragma unroll 1
    for (int x = w; x < NTP; x += NW) {
      const int i = tri_row_of(x, false), j = tri_col_of(x, false);
      const T* pu = sU + RT::at(16 * j + c, 0, 4 * g);
      const T* pr = sR + RT::at(16 * i + c, 0, 4 * g);
      const T* po = sdO + RT::at(16 * i + c, 0, 4 * g);
      f32x4 accA = zero4(), accP = zero4();
      for (int vp = 0; vp < NJT / 2; ++vp) {
        const quad u0 = Qd::ld(pu + 32 * vp), u1 = Qd::ld(pu + 32 * vp + 16);
        accA = Qd::mma32(u0, u1, Qd::ld(pr + 32 * vp), Qd::ld(pr + 32 * vp + 16), accA);
        accP = Qd::mma32(u0, u1, Qd::ld(po + 32 * vp), Qd::ld(po + 32 * vp + 16), accP);
      }
      for (int e = 0; e < 4; ++e) {
        accA[e] = (i > j || 4 * g + e < c) ? accA[e] : 0.0f;
        accP[e] = (i > j || 4 * g + e <= c) ? accP[e] : 0.0f;
      }
      Qd::st(sdA + x * ST::N + ST::at(c, 4 * g), Qd::cvt(accA));
      Qd::st(sdP + x * ST::N + ST::at(c, 4 * g), Qd::cvt(accP));
    }
    f32x4 y[NB], dQ[NB], dKi[NB];
    float dgs = 0.0f;   // sum_v dM[v][j] S'[v][j] for j = 16 w + c
    for (int tt = 0; tt < NB; ++tt) {
      y[tt] = zero4();
      dQ[tt] = zero4();
      dKi[tt] = zero4();
    }
    for (int vp = 0; vp < NJT / 2; ++vp) {
      CARVE_SEQ();
      const quad a0 = RT::tr(sdM, 32 * vp, 16 * w, g, c), a1 = RT::tr(sdM, 32 * vp + 16, 16 * w, g, c);
      const quad s0 = sS[2 * vp], s1 = sS[2 * vp + 1];
      for (int tt = 0; tt < NB; ++tt) {
        const int o0 = RT::at(16 * tt + c, 32 * vp, 4 * g), o1 = RT::at(16 * tt + c, 32 * vp + 16, 4 * g);
        y[tt] = Qd::mma32(s0, s1, Qd::ld(sR + o0), Qd::ld(sR + o1), y[tt]);
        dQ[tt] = Qd::mma32(s0, s1, Qd::ld(sdO + o0), Qd::ld(sdO + o1), dQ[tt]);
        dKi[tt] = Qd::mma32(a0, a1, Qd::ld(sU + o0), Qd::ld(sU + o1), dKi[tt]);
      }
      const f32x4 x0 = Qd::f32(a0), x1 = Qd::f32(a1), y0 = Qd::f32(s0), y1 = Qd::f32(s1);
      for (int e = 0; e < 4; ++e) dgs += x0[e] * y0[e] + x1[e] * y1[e];
    }
    dgs += __shfl_xor(dgs, 16);
    dgs += __shfl_xor(dgs, 32);
    // wave 0 waits for the next chunk's record; every wave reads the outcome
    // from LDS after the barrier
    if (wait_ch >= 0 && w == 0) wait_ready(wait_ch, timed_out);
    __syncthreads();

    // ---- B3: pair terms, gate gradients ------------------------------------------
    fresh();
    // gradients of the token rows go to LDS first (dv, dk over dO and U, dz_w,
    // dz_b and later dq over dM and R) and out in whole rows from there: stores
    // of 16 rows for 32 bytes each held up every wave behind the CU's memory
    // pipeline
    for (int tt = 0; tt < NB; ++tt) {
      Qd::st(sdO + RT::at(16 * tt + c, 16 * w, 4 * g), dvT[tt]);
      if constexpr (!SW) Qd::st(sdM + RT::at(16 * tt + c, 16 * w, 4 * g), dzwT[tt]);
    }
    if (wait_ch >= 0) after_wait(s, timed_out);
    // the next block (at the call's first block there is none: this one's data is
    // read again then, so that p is written on every path)
    int pch = ch, pm = next_m, pwide = 0;
    if constexpr (NEXT) {
      const int nctl = reinterpret_cast<const int*>(smem + lay.Ctl)[0];   // wide bits of the awaited chunk, or -1
      if (next_m >= 0) {
        pwide = (wide >> next_m) & 1;
      } else if (wait_ch >= 0) {
        pch = wait_ch;
        pm = mpc - 1;
        pwide = nctl > 0 ? (nctl >> pm) & 1 : 0;
      } else {
        pm = 0;
      }
    }
    // operands of B4 and B5, loaded ahead of this step's stores (a wait for a
    // load also waits for every store issued before it)
    quad qT[NB];
    for (int tt = 0; tt < NB; ++tt)
      qT[tt] = TILE ? tp.q : rc.template ld<quad>(cr.Q + (tile0 + tt) * NT * QB, tid * QB);
    quad tauq[NVS][(NB + NTW - 1) / NTW], fV[NVS][NJT];
    for (int k = 0; k < NVS; ++k)
      for (int jt = 0; jt < NJT; ++jt) fV[k][jt] = Qd::ld(opnd + ((size_t)(k * NJT + jt) * NT + tid) * 4);
    for (int k = 0; k < NVS; ++k)
      for (int u = 0; u < (NB + NTW - 1) / NTW; ++u) {
        const int tt = w / NRW + u * NTW;
        if constexpr (TILE) tauq[k][u] = tp.tau[k];
        else if (tt < NB) tauq[k][u] = load_tau(rc, tile0 + tt, w % NRW + k * NRW);
      }
    f32x4 km[NB];
    f32x4 dgg;
    {
      f32x4 ds = zero4();
      for (int tt = 0; tt < NB; ++tt) {
        km[tt] = Qd::f32(Qd::ld(sKi + RT::at(16 * tt + c, 16 * w, 4 * g)));
        ds += km[tt] * dKi[tt];
      }
      for (int i = 0; i < 4; ++i) dgg[i] = __shfl(dgs, 4 * g + i) + row_bcast15(row_scan(ds[i]));
    }
    {
      quad kiT[NB], ktT[NB], qtT[NB];
      for (int tt = 0; tt < NB; ++tt) {
        kiT[tt] = RT::tr(sKi, 16 * tt, 16 * w, g, c);
        ktT[tt] = RT::tr(sKt, 16 * tt, 16 * w, g, c);
        qtT[tt] = RT::tr(sQt, 16 * tt, 16 * w, g, c);
      }
      for (int i = 0; i < NB; ++i)
        for (int j = 0; j <= i; ++j) {
          const T* ta = sdA + tri_incl(i, j) * ST::N;
          const T* tp = sdP + tri_incl(i, j) * ST::N;
          y[i] = Qd::mma16(kiT[j], Qd::ld(ta + ST::at(c, 4 * g)), y[i]);
          dQ[i] = Qd::mma16(kiT[j], Qd::ld(tp + ST::at(c, 4 * g)), dQ[i]);
          dKi[j] = Qd::mma32(ktT[i], qtT[i], ST::tr(ta, g, c), ST::tr(tp, g, c), dKi[j]);
        }
    }
    // elementwise, last tile first: lane (g, c) holds j = 16 w + 4 g + i, t = 16 tt + c
    {
      f32x4 nxt_in = zero4(), dl_in = zero4();   // from the tile after: y Kh of its first token, its dl
      for (int tt = NB - 1; tt >= 0; --tt) {
        const f32x4 ktM = Qd::f32(Qd::ld(sKt + RT::at(16 * tt + c, 16 * w, 4 * g)));
        const f32x4 qtM = Qd::f32(Qd::ld(sQt + RT::at(16 * tt + c, 16 * w, 4 * g)));
        const float bt = sBeta[16 * tt + c];
        const f32x4 sg = Qd::f32(sig[tt]);
        f32x4 dgv, dzb, dkv;
        float pb = 0.0f;
        for (int i = 0; i < 4; ++i) {
          const float Ei = fast_rcp(E[tt][i]);
          // e^{lam_{t-1} - rho}; before the block's first token e^{-rho} = 1 / E of the last
          const float fill = tt > 0 ? row_bcast15(E[tt > 0 ? tt - 1 : 0][i]) : fast_rcp(row_bcast15(E[NB - 1][i]));
          const float Ep = row_shr1(E[tt][i], fill);
          const float yk = y[tt][i] * ktM[i];
          float dlam = dQ[tt][i] * qtM[i] - dKi[tt][i] * km[tt][i] + row_shl1(yk, nxt_in[i]);
          nxt_in[i] = row_bcast0(yk);
          if (tt == NB - 1 && c == 15) dlam += dgg[i];
          const float dl = row_suffix(dlam) + dl_in[i];
          dl_in[i] = row_bcast0(dl);
          dgv[i] = dl;
          dzb[i] = -dl * sg[i];
          const float yp = y[tt][i] * Ep;
          pb += km[tt][i] * E[tt][i] * yp;
          dkv[i] = bt * yp + dKi[tt][i] * Ei;
          dQ[tt][i] *= E[tt][i];
        }
        Qd::st(sU + RT::at(16 * tt + c, 16 * w, 4 * g), Qd::cvt(dkv));
        if constexpr (GATED) {
          // through Eq. decay_gate: df = dg (-exp(A)) sigmoid(f + tau_f); dA and
          // dtau collect dg g and df
          const f32x4 fv = Qd::f32(Qd::ld(reinterpret_cast<const T*>(a.f) + bh0 + e0(tt)));
          const f32x4 na = *reinterpret_cast<const f32x4*>(gate(0)), tf = *reinterpret_cast<const f32x4*>(gate(1));
          f32x4 dfv;
          for (int i = 0; i < 4; ++i) {
            float sp, sgf;
            softplus_sigmoid(fv[i] + tf[i], sp, sgf);
            dfv[i] = dgv[i] * na[i] * sgf;
            s.gA[i] += dgv[i] * na[i] * sp;
            s.gT[i] += dfv[i];
          }
          Qd::st(reinterpret_cast<T*>(a.df) + bh0 + e0(tt), Qd::cvt(dfv));
        } else {
          *reinterpret_cast<f32x4*>(a.dg + bh0 + e0(tt)) = dgv;
        }
        Qd::st(sR + RT::at(16 * tt + c, 16 * w, 4 * g), Qd::cvt(dzb));
        // dbeta, key part: sum over j of Kt y with Kt = k e^{lam_{t-1} - rho}, k = Ki E
        pb += __shfl_xor(pb, 16);
        pb += __shfl_xor(pb, 32);
        if (g == 0) sDbeta[16 * tt + c] += pb;
      }
    }
    __syncthreads();

    // ---- B4: dtau^T (rows r, column t) and dY = dtau (1 - tau^2) -> sdY[t][r] -------
    fresh();
    // operands of B5 and of the glue, ahead of the next block's data
    quad FT[NRT];
    if constexpr (TILE) {
      for (int rt = 0; rt < NRT; ++rt) FT[rt] = tp.FT[rt];
    } else {
      load_fold(fU, FT, ch);
    }
    for (int k = 0; k < NVS; ++k)
      for (int u = 0; u < (NB + NTW - 1) / NTW; ++u) {
        const int rt = w % NRW + k * NRW, tt = w / NRW + u * NTW;
        if (tt < NB) {
          const T* src = rt < NRB ? sR : sdM;   // dz_b or dz_w
          f32x4 acc = zero4();
          for (int jp = 0; jp < NJT / 2; ++jp)
            acc = Qd::mma32(fV[k][2 * jp], fV[k][2 * jp + 1], Qd::ld(src + RT::at(16 * tt + c, 32 * jp, 4 * g)),
                            Qd::ld(src + RT::at(16 * tt + c, 32 * jp + 16, 4 * g)), acc);
          const f32x4 tau = Qd::f32(tauq[k][u]);
          for (int i = 0; i < 4; ++i) acc[i] *= 1.0f - tau[i] * tau[i];
          Qd::st(sdY + RY::at(16 * tt + c, 16 * rt, 4 * g), Qd::cvt(acc));
        }
      }
    store_rows<NB>(a.dv, sdO, t0);
    store_rows<NB>(a.dk, sU, t0);
    store_rows<NB>(a.dbx, sR, t0);
    if constexpr (!SW) store_rows<NB>(a.dwx, sdM, t0);
    // the next block's (tile's) data, on its way during B5 and the glue
    if constexpr (NEXT) {
      load_tiles(p, pch, pm);
      load_scalars(p, pch, pm, pwide);
      load_uo(p, pch, pm);
    } else {
      load_tile(tp, ch, tile0 - 1);
    }
    // dbeta (and the scalar write gate's dwx): the waves' partials in order
    if (w == NW - 1)
      for (int t = tid & 63; t < W; t += 64) {
        float sb = 0.0f, sw = 0.0f;
        for (int ww = 0; ww < NW; ++ww) sb += ldf(lay.Dbeta)[ww * W + t];
        reinterpret_cast<T*>(a.dbeta)[bh1 + (size_t)(t0 + t) * H] = (T)sb;
        if constexpr (SW) {
          for (int ww = 0; ww < NW; ++ww) sw += ldf(lay.Dwx)[ww * W + t];
          reinterpret_cast<T*>(a.dwx)[bh1 + (size_t)(t0 + t) * H] = (T)sw;
        }
      }
    __syncthreads();

    // ---- B5: dF += dY^T q, dq = dQt E + dY F (key tile w) ------------------------------
    fresh();
    // dF starts from that of the chunk's later blocks, parked in its record
    // (a block's tiles hand it on in registers)
    if (!TILE || sub == NBK - 1)
      for (int rt = 0; rt < NRT; ++rt) dF[rt] = zero4();
    if (16 * (tile0 + NB) < L && (!TILE || sub == NBK - 1)) {
      const float* dFr = reinterpret_cast<const float*>(rec_of(ch) + cr.dF) + (size_t)(16 * w + c) * RF + 4 * g;
      for (int rt = 0; rt < NRT; ++rt) dF[rt] = *reinterpret_cast<const f32x4*>(dFr + 16 * rt);
      // (waited for here: a load still pending where the two paths join would
      // make both of them wait, for the next block's data too)
      for (int rt = 0; rt < NRT; ++rt) arrived(dF[rt]);
    }
    if constexpr (!TILE)
      for (int rt = 0; rt < NRT; ++rt) arrived(fU[rt]);
    for (int rt = 0; rt < NRT; ++rt) {
      if constexpr (NB == 1) {
        dF[rt] = Qd::mma16(RY::tr(sdY, 0, 16 * rt, g, c), qT[0], dF[rt]);
      } else {
        for (int tp = 0; tp < NB / 2; ++tp)
          dF[rt] = Qd::mma32(RY::tr(sdY, 32 * tp, 16 * rt, g, c), RY::tr(sdY, 32 * tp + 16, 16 * rt, g, c), qT[2 * tp],
                               qT[2 * tp + 1], dF[rt]);
      }
    }
    for (int tt = 0; tt < NB; ++tt) {
      f32x4 acc = dQ[tt];
      for (int rp = 0; rp < NRT / 2; ++rp)
        acc = Qd::mma32(FT[2 * rp], FT[2 * rp + 1], Qd::ld(sdY + RY::at(16 * tt + c, 32 * rp, 4 * g)),
                        Qd::ld(sdY + RY::at(16 * tt + c, 32 * rp + 16, 4 * g)), acc);
      Qd::st(sR + RT::at(16 * tt + c, 16 * w, 4 * g), Qd::cvt(acc));
    }
    for (int rt = 0; rt < NRT; ++rt) arrived(dF[rt]);
    if (tile0 > 0 && (!TILE || sub == 0)) park_dF(dF, ch);
  }
  // NB * 16 token rows of a tile to the rows from t0 on of a token tensor
  template <int NB>
  __device__ __forceinline__ void store_rows(void* dst, const T* tile, int t0) const {
    T* d = reinterpret_cast<T*>(dst) + bh0 + (size_t)t0 * rs;
    constexpr int N = 16 * NB * D / VEC;
    for (int u = 0; u < (N + NT - 1) / NT; ++u) {
      const int x = tid + u * NT;
      if (N % NT != 0 && x >= N) break;
      const int row = x / (D / VEC), k = x % (D / VEC);
      *reinterpret_cast<u32x4_t*>(d + row * rs + k * VEC) = unstage_vec<T, D>(tile, row, k);
    }
  }
  // dF of a chunk in its record, as [j][r] (a lane holds four consecutive r of
  // one j: one 16-byte store per tile)
  __device__ __forceinline__ void park_dF(const f32x4 (&dF)[NRT], int ch) const {
    float* dFr = reinterpret_cast<float*>(const_cast<char*>(rec_of(ch)) + cr.dF) + (size_t)(16 * w + c) * RF + 4 * g;
    for (int rt = 0; rt < NRT; ++rt) *reinterpret_cast<f32x4*>(dFr + 16 * rt) = dF[rt];
  }

  // wave 0: wait until chunk need's flag is raised (the record is read with
  // agent-scope loads, RecBuf, so no cache is invalidated here); Ctl[0] = its wide bits, or
  // -1 if the bound ran out (or had before)
  __device__ __forceinline__ void wait_ready(int need, bool timed_out) const {
    int* ctl = reinterpret_cast<int*>(smem + lay.Ctl);
    const int* rdy = ready + (size_t)bh * nch + need;
    int v = 0;
    if (!timed_out)
      for (int n = 0; n < a.wait_limit; ++n) {
        v = __hip_atomic_load(rdy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v != 0) break;
        __builtin_amdgcn_s_sleep(2);
      }
    if (lane == 0) ctl[0] = v != 0 ? v >> 1 : -1;
  }
  // every wave, after the barrier that follows wait_ready
  __device__ __forceinline__ void after_wait(State& s, bool& timed_out) const {
    const int v = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(smem + lay.Ctl)[0]);
    if (v < 0 && !timed_out) {
      timed_out = true;
      const float n = __builtin_nanf("");
      for (int jt = 0; jt < NJT; ++jt) s.dS[jt] = f32x4{n, n, n, n};
      if (tid == 0) __hip_atomic_store(timeout_word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  const int* ready;
  int* timeout_word;
  int* pos;

  // dS += [Ub; Uw]^T dF at a chunk start; dF is parked in the chunk record for
  // d[Ub; Uw] += dF S_hat^T (carve_bwd_param_kernel).  dF enters the product as
  // a high and a low part (bf16) so that its f32 accumulation is not rounded
  // away.  Reads dY's step as finished only after its barrier.
  __device__ __forceinline__ void glue(State& s, f32x4 (&dF)[NRT], const quad (&fU)[NRT], int ch) {
    fresh();
    T* sh = lds(lay.U);
    T* sl = sh + D * LDF;
    for (int rt = 0; rt < NRT; ++rt) {
      const quad hi = Qd::cvt(dF[rt]);
      Qd::st(sh + df_at(16 * w + c, 16 * rt + 4 * g), hi);
      if constexpr (SPLIT) Qd::st(sl + df_at(16 * w + c, 16 * rt + 4 * g), Qd::cvt(dF[rt] - Qd::f32(hi)));
    }
    park_dF(dF, ch);
    __syncthreads();
    for (int jt = 0; jt < NJT; ++jt) {
      CARVE_SEQ();
      f32x4 acc = s.dS[jt];
      for (int rp = 0; rp < NRT / 2; ++rp) {
        const int o0 = df_at(16 * jt + c, 32 * rp + 4 * g), o1 = df_at(16 * jt + c, 32 * rp + 16 + 4 * g);
        acc = Qd::mma32(Qd::ld(sh + o0), Qd::ld(sh + o1), fU[2 * rp], fU[2 * rp + 1], acc);
        if constexpr (SPLIT) acc = Qd::mma32(Qd::ld(sl + o0), Qd::ld(sl + o1), fU[2 * rp], fU[2 * rp + 1], acc);
      }
      s.dS[jt] = acc;
    }
  }

  __device__ __forceinline__ void run() {
    // running: the recompute may follow this adjoint
    if (tid == 0) __hip_atomic_store(pos, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // operand quads of the parameters, written once to this workgroup's part of
    // the workspace in thread order and read back where they are used (each
    // thread its own; from cache): V^T of the wave's dtau tiles (lane (g, c):
    // V[16 jt + 4 g + e][16 rt' + c], rows past R zero) and [Ub; Uw] of the glue
    // (lane (g, c): U[16 rt + 4 g + e][16 w + c]).  Held in registers they would
    // push the block's tiles into scratch.
    for (int k = 0; k < NVS; ++k) {
      const int rt = w % NRW + k * NRW;
      const float* src = rt < NRB ? a.Vb : a.Vw;
      const int r = 16 * (rt % NRB) + c;
      for (int jt = 0; jt < NJT; ++jt) {
        f32x4 t;
        for (int e = 0; e < 4; ++e) t[e] = r < R ? src[(16 * jt + 4 * g + e) * R + r] : 0.0f;
        Qd::st(opnd + ((size_t)(k * NJT + jt) * NT + tid) * 4, Qd::cvt(t));
      }
    }
    for (int rt = 0; rt < NRT; ++rt) {
      const float* src = rt < NRB ? a.Ub : a.Uw;
      f32x4 t;
      for (int e = 0; e < 4; ++e) {
        const int r = 16 * (rt % NRB) + 4 * g + e;
        t[e] = r < R ? src[r * D + 16 * w + c] : 0.0f;
      }
      Qd::st(opnd + ((size_t)(NVS * NJT + rt) * NT + tid) * 4, Qd::cvt(t));
    }
    if constexpr (GATED)
      for (int e = 0; e < 4; ++e) {
        gate(0)[e] = -expf(a.A[h * D + 16 * w + 4 * g + e]);
        gate(1)[e] = a.tau_f[h * D + 16 * w + 4 * g + e];
      }
    State s;
    const size_t soff = (size_t)bh * D * D;
    for (int jt = 0; jt < NJT; ++jt)
      s.dS[jt] = a.dS_T ? gload4(a.dS_T + soff + (16 * w + c) * D + 16 * jt + 4 * g) : zero4();
    s.gA = s.gT = zero4();
    Pre p;
    TilePre tp;
    bool timed_out = false;
    int dq_t0 = -1;   // first token of the block whose dq rows are in LDS
    if (w == 0) wait_ready(nch - 1, false);
    __syncthreads();
    after_wait(s, timed_out);
    {
      const int ctl = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(smem + lay.Ctl)[0]);
      load_tiles(p, nch - 1, mpc - 1);
      load_scalars(p, nch - 1, mpc - 1, ctl > 0 && ((ctl >> (mpc - 1)) & 1));
      load_uo(p, nch - 1, mpc - 1);
    }

#pragma unroll 1
    for (int ch = nch - 1; ch >= 0; --ch) {
      const int ctl = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(smem + lay.Ctl)[0]);
      const int wide = ctl > 0 ? ctl : 0;
      if (tid == 0) __hip_atomic_store(pos, 1 + nch - ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      f32x4 dF[NRT];
      quad fU[NRT];
#pragma unroll 1
      for (int m = mpc - 1; m >= 0; --m) {
        const int wait_ch = m == 0 ? ch - 1 : -1;
        load_vals(p, ch, m);   // (first used in the middle of B1)
        // (the last readers of the other regions were before B5; U and dO are
        // read by the glue)
        put_tiles(p);
        __syncthreads();
        if (dq_t0 >= 0) store_rows<NBK>(a.dq, lds(lay.R), dq_t0);
        put_uo(p);
        __syncthreads();
        if (NBK == 1 || !((wide >> m) & 1)) {
          block<NBK, true>(s, p, tp, dF, fU, ch, m * NBK, 0, wait_ch, timed_out, m - 1, wide);
        } else if constexpr (NBK > 1) {
          // tile by tile, from the same data in LDS; a tile's reference, gates and
          // values are loaded during the one after it
          load_tile(tp, ch, m * NBK + NBK - 1);
          load_fold(fU, tp.FT, ch);
#pragma unroll 1
          for (int i = NBK - 1; i > 0; --i) {
            block<1, false>(s, p, tp, dF, fU, ch, m * NBK + i, i, -1, timed_out, -1, 0);
            put_gam(tp.gam);   // (last read in B1)
            __syncthreads();
          }
          block<1, true>(s, p, tp, dF, fU, ch, m * NBK, 0, wait_ch, timed_out, m - 1, wide);
          // nothing of this path is pending where it joins the other one (the
          // join would make that one wait for the next block's data otherwise)
          vm_wait_all();
        }
        dq_t0 = ch * L + m * W;
        if (m == 0) glue(s, dF, fU, ch);
      }
    }
    __syncthreads();
    if (dq_t0 >= 0) store_rows<NBK>(a.dq, lds(lay.R), dq_t0);
    if constexpr (GATED) {
      // the lanes' sums over their tokens, reduced over the 16 lanes of a row
      // (all tokens of a tile) and written by lane c = 0, one owner per channel
      for (int i = 0; i < 4; ++i) {
        s.gA[i] = row_suffix(s.gA[i]);
        s.gT[i] = row_suffix(s.gT[i]);
      }
      if (c == 0) {
        float* dst = a.partG + (size_t)bh * 2 * D + 16 * w + 4 * g;
        *reinterpret_cast<f32x4*>(dst) = s.gA;
        *reinterpret_cast<f32x4*>(dst + D) = s.gT;
      }
    }
    if (a.dS0) {
      float* dst = a.dS0 + soff + (16 * w + c) * D + 4 * g;
      for (int jt = 0; jt < NJT; ++jt) *reinterpret_cast<f32x4*>(dst + 16 * jt) = s.dS[jt];
    }
  }

  __device__ __forceinline__ Adjoint(const BwdArgs& a_, int bh_, char* smem_, const int* ready_, int* timeout_, int* pos_)
      : a(a_), bh(bh_), smem(smem_), ready(ready_), timeout_word(timeout_), pos(pos_) {
    tid = threadIdx.x;
    lane = tid & 63;
    w = __builtin_amdgcn_readfirstlane(tid >> 6);
    g = lane >> 4;
    c = lane & 15;
    H = a.H;
    L = a.L;
    R = a.R;
    nch = a.T / L;
    mpc = L / W;
    rs = H * D;
    h = bh % H;
    cr = chunk_rec<T, D>(L, RF, NBK);
    bh0 = ((size_t)(bh / H) * a.T * H + h) * D;
    bh1 = (size_t)(bh / H) * a.T * H + h;
    recb = reinterpret_cast<const char*>(a.rec) + (size_t)bh * nch * cr.total;
    opnd = reinterpret_cast<T*>(reinterpret_cast<char*>(a.opnd) + (size_t)bh * adj_opnd_bytes(D, 2 * RP, sizeof(T)));
  }
};

// Chunk recompute and adjoint in one grid of nrec + B*H workgroups.  Roles go
// by arrival: each workgroup draws a ticket from the counter in sync; the first
// nrec tickets recompute, the rest run the adjoint of (batch, head) ticket -
// nrec.  A workgroup with a recompute ticket is already running and waits only
// for a bounded time, so every flag an adjoint workgroup waits for is raised in
// finite time whatever order the hardware dispatches the grid in.  With lead >
// 0 a recompute workgroup starts a chunk only once the adjoint of its (batch,
// head) has started the chunk lead places before it (a bounded wait,
// kPresentSpinLimit and kLeadSpinLimit): records are then written shortly before
// they are read, and the recompute's stores do not all come at once.
template <typename T, int D, int RP, int VAR, int NB>
__global__ void __launch_bounds__(bwd_threads(D)) __attribute__((amdgpu_waves_per_eu(1, 2)))
carve_bwd_fused_kernel(FwdArgs f, BwdArgs a, int nrec, int* sync, int lead) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nbh = a.B * a.H, nch = a.T / a.L;
  if (threadIdx.x == 0)
    reinterpret_cast<int*>(smem)[0] =
        __hip_atomic_fetch_add(sync + sync_ticket(nbh, nch), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(smem)[0]);
  __syncthreads();
  if (ticket < nrec) {
    rec_run<T, D, RP, VAR, NB>(f, ticket, nrec, sync, lead, smem);
  } else {
    const int bh = ticket - nrec;
    Adjoint<T, D, RP, VAR, NB>(a, bh, smem, sync, sync + sync_timeout_word(nbh, nch), sync + sync_adjoint_pos(nbh, nch) + bh)
        .run();
  }
}

// ---------------------------------------------------------------------------
// host-side launch
// ---------------------------------------------------------------------------
template <typename T, int D, int RP, int VAR, int NB>
static int launch_fused_t(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, hipStream_t stream) {
  constexpr size_t lds = fused_lds<T, D, RP, VAR, NB>();
  if constexpr (lds > kMaxLdsBytes) {
    return CARVE_ERR_UNSUPPORTED;
  } else {
    auto kern = carve_bwd_fused_kernel<T, D, RP, VAR, NB>;
    static bool attr_set = false;  // per instantiation
    if (!attr_set) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds) != hipSuccess)
        return CARVE_ERR_HIP;
      attr_set = true;
    }
    // the adjoint workgroups take B*H compute units (one workgroup per CU: the
    // LDS layout); the recompute gets the rest, or the whole device first when
    // fewer than a quarter would remain
    const int nbh = a.B * a.H;
    const long long nitems = (long long)nbh * (a.T / a.L);
    long long nrec = cus - nbh;
    if (nrec < cus / 4) nrec = cus;
    if (nrec > nitems) nrec = nitems;
    if (nrec < 1) nrec = 1;
    // pace the recompute only when every workgroup of the grid can be resident
    // at once (one per compute unit), so that the adjoints it follows run unless
    // other work holds compute units
    const int lead = nrec + nbh <= cus ? recompute_lead(a.L) : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)(nrec + nbh)), dim3(bwd_threads(D)), lds, stream, f, a, (int)nrec, sync,
                       lead);
    return hipGetLastError() == hipSuccess ? CARVE_OK : CARVE_ERR_HIP;
  }
}

template <typename T, int D, int RP, int VAR>
static int launch_fused_l(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, int NB, hipStream_t s) {
  if (NB == 1) return launch_fused_t<T, D, RP, VAR, 1>(f, a, sync, cus, s);
  if constexpr (sizeof(T) == 2) {   // f32: one-tile blocks only (bwd_lds_bytes)
    if (NB == 2) return launch_fused_t<T, D, RP, VAR, 2>(f, a, sync, cus, s);
    if (NB == 4) return launch_fused_t<T, D, RP, VAR, 4>(f, a, sync, cus, s);
  }
  return CARVE_ERR_UNSUPPORTED;
}

template <typename T, int VAR>
static int launch_fused_d(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, int D, int NB, hipStream_t s) {
  if (a.RP == 32) {
    if (D == 32) return launch_fused_l<T, 32, 32, VAR>(f, a, sync, cus, NB, s);
    if (D == 64) return launch_fused_l<T, 64, 32, VAR>(f, a, sync, cus, NB, s);
    if constexpr (sizeof(T) == 2)
      if (D == 128) return launch_fused_l<T, 128, 32, VAR>(f, a, sync, cus, NB, s);
  } else if (a.RP == 64) {
    if (D == 32) return launch_fused_l<T, 32, 64, VAR>(f, a, sync, cus, NB, s);
    if constexpr (sizeof(T) == 2)
      if (D == 64) return launch_fused_l<T, 64, 64, VAR>(f, a, sync, cus, NB, s);
  }
  return CARVE_ERR_UNSUPPORTED;
}

template <int VAR>
int launch_bwd_fused_var(const FwdArgs& f, const BwdArgs& a, int* sync, int cus, int dtype, int D, int NB,
                         hipStream_t s) {
  if (dtype == CARVE_BF16) return launch_fused_d<bf16_t, VAR>(f, a, sync, cus, D, NB, s);
  return launch_fused_d<float, VAR>(f, a, sync, cus, D, NB, s);
}

}  // namespace carve

// carve_rec.h -- chunk recompute of the CARVE backward on gfx950.
//
// rec_run() recomputes gate chunks of single (batch, head) pairs from their
// start states (S_chunks, written by the forward) and writes, per chunk, the
// record that the adjoint reads (ChunkRec).  Every chunk is independent, so the
// recompute is chunk-parallel.  Wave w of the workgroup owns the 16-wide tile w
// of the value axis and the 16-wide tile w of the key axis:
//   * the state lives in registers as S^T tiles (rows = key index j, columns =
//     the wave's 16 value rows v), in the matrix-core result layout;
//   * everything on the value side (predictions, WY solve, state update) is
//     wave-local;
//   * the key-side gate arithmetic (erase gate, log retention, its prefix sums
//     and the decayed keys/queries) runs on the wave's key tile.
//
// Per gate chunk with start state S_hat (Eq. content_readout):
//   F = [Ub; Uw] S_hat                         (fold, once per chunk)
//   tau = tanh(q F^T), z_b = bx + tau_b Vb^T, z_w = wx + tau_w Vw^T
//   l = g - softplus(z_b) = log(exp(g) (1 - b)), w = sigmoid(z_w)
// and then, for consecutive WY blocks of NB 16-token tiles (Sec. 6.2 applied
// block by block; every block of the chunk uses the same F), with lam = prefix
// sums of l inside the block (lam_{-1} = 0), the block reference rho =
// lam_end / 2 per key channel (the middle of the block's log-retention range),
// state S at the block start and u the WY "pseudo values":
//   Kh_t = beta_t k_t e^{lam_{t-1} - rho},  Ki_s = k_s e^{rho - lam_s},  Qt_t = q_t e^{lam_t - rho}
//   S' = S diag(e^{rho})
//   A_ts = Kh_t . Ki_s (s < t),  P_ts = Qt_t . Ki_s (s <= t)
//   T_ii = (I + A_ii)^{-1} per 16-token tile,  R_t = beta_t w_t * v_t - S' Kh_t
//   u = (I + A)^{-1} R                  (blocked over the tiles)
//   S <- (S' + sum_s u_s Ki_s^T) diag(e^{rho})     (only where a block follows)
// which is the recurrence of Eq. carve_state rewritten exactly (every pair of
// factors multiplies to e^{lam_a - lam_b} with a >= b).  beta is folded into
// the key operand, so that the adjoint has one rounded operand for A and for
// the prediction.  No factor exceeds e^{|lam_end| / 2}.
//
// A block in which some key channel decays by more than e^{-kBwdWideLog} is
// evaluated tile by tile instead: lam, rho and the state run per 16-token tile,
// and the adjoint walks the block's tiles as blocks of one tile.  The choice is
// a vote of the workgroup and goes to the adjoint with the chunk's ready flag.
//
// With the scalar write gate (kVarScalarW) F = Ub S_hat has R rows and
// w_t = sigmoid(wx_t) is one scalar per token and head, staged with beta.
// With the input activations (kVarAct) q, k, v arrive raw: the rows of q and k
// are staged as SiLU(raw) / |SiLU(raw)|, v as SiLU(raw).
//
// What bounds it: a dependent sequence of seven barrier-separated steps on one
// workgroup per compute unit (the LDS layout), two waves per SIMD; the token
// rows and the start state of the next block are loaded into registers while
// the current one runs, and a chunk's flag is raised only after the next
// chunk's first wait, so that no step waits for the stores just issued.
//
// Precondition (not checked): within any 16-token tile the log retention
// summed over the tile stays above about -170 per key channel, so that
// e^{|tile log retention| / 2} is finite in f32 and bf16.
#pragma once
#include "carve_kernels.h"

namespace carve {

// 16-byte vectors x of [rows][D] token rows staged into a RowTile
// (L2: raw q or k rows, staged as SiLU(raw) / |SiLU(raw)|; SILU: as SiLU(raw)).
// A row's vectors sit in consecutive lanes of one wave.
template <typename T, int D, bool L2, bool SILU>
__device__ __forceinline__ void stage_vec(T* dst, int x, u32x4_t r) {
  constexpr int VEC = 16 / sizeof(T);
  if constexpr (L2) r = act_chunk<T>(r, act_row_inv_norm<T, D / VEC>(r));
  if constexpr (SILU) r = act_chunk<T>(r, 1.0f);
  const int row = x / (D / VEC), k = x % (D / VEC);
  if constexpr (sizeof(T) == 2) {
    // the vector's quads 2k, 2k + 1 go to quads (2k, 2k + 1) ^ h
    const int h = RowTile<T, D>::sw(row) >> 2;
    if (h & 1) r = u32x4_t{r[2], r[3], r[0], r[1]};
    *reinterpret_cast<u32x4_t*>(dst + row * RowTile<T, D>::LD + (((2 * k) ^ (h & ~1)) * 4)) = r;
  } else {
    *reinterpret_cast<u32x4_t*>(dst + row * RowTile<T, D>::LD + k * VEC) = r;
  }
}

// 16-byte vector k of row `row` of a RowTile
template <typename T, int D>
__device__ __forceinline__ u32x4_t unstage_vec(const T* src, int row, int k) {
  constexpr int VEC = 16 / sizeof(T);
  if constexpr (sizeof(T) == 2) {
    const int h = RowTile<T, D>::sw(row) >> 2;
    const u32x4_t r = *reinterpret_cast<const u32x4_t*>(src + row * RowTile<T, D>::LD + (((2 * k) ^ (h & ~1)) * 4));
    return (h & 1) ? u32x4_t{r[2], r[3], r[0], r[1]} : r;
  } else {
    return *reinterpret_cast<const u32x4_t*>(src + row * RowTile<T, D>::LD + k * VEC);
  }
}

// Recompute of the items first, first + stride, ... < nitems: item i is chunk
// nch - 1 - i / (B*H) of (batch, head) i % (B*H) (latest chunks first, the order
// in which the adjoint needs them).  sync: the synchronisation area (ready
// flags, adjoint positions); with lead > 0 an item is started only once the
// adjoint of its (batch, head) has started the chunk lead places before it.  A
// workgroup whose wait runs out follows no adjoint any more, so that waiting
// costs it one bound in all and not one per item (other streams' work may hold
// the compute units that the adjoints would take).
// smem: the workgroup's dynamic LDS (RecLds layout).
// Bounds of that wait, in polls of a few hundred cycles: for an adjoint that has
// not begun (2^8, about 100 us, many times a launch's own spread), and for one
// that has (2^16, tens of milliseconds; it waits for nothing but other chunks'
// recompute).
constexpr int kPresentSpinLimit = 1 << 8;
constexpr int kLeadSpinLimit = 1 << 16;

template <typename T, int D, int RP, int VAR, int NB>
__device__ __forceinline__ void rec_run(const FwdArgs& a, const int first, const int stride, int* sync, int lead,
                                        char* smem) {
  typedef Quad<T> Qd;
  typedef typename Qd::q quad;
  typedef RowTile<T, D> RT;
  typedef SmallTile<T> ST;
  constexpr bool GATED = (VAR & kVarGated) != 0;
  constexpr bool SW = (VAR & kVarScalarW) != 0;
  constexpr bool ACT = (VAR & kVarAct) != 0;
  constexpr int NT = fwd_threads(D);
  constexpr int NW = NT / 64;          // waves == 16-wide tiles of the key / value axis
  constexpr int NJT = D / 16;
  constexpr int W = 16 * NB;           // tokens of a block
  constexpr int RF = fold_rows(RP, VAR);
  constexpr int NRT = RF / 16, NRB = RP / 16;
  typedef RowTile<T, RF> RTau;
  constexpr int VEC = 16 / sizeof(T);
  constexpr unsigned QB = 4 * sizeof(T);             // bytes of a quad
  constexpr int NVX = W * D / VEC;                   // 16-byte vectors of one [W][D] tile
  constexpr int NXV = (NVX + NT - 1) / NT;           // per thread
  constexpr int NTA = tiles_a(NB), NTP = tiles_p(NB);
  constexpr int NDW = NB < NW ? NB : NW;             // waves with a diagonal inverse
  constexpr int NOW = NW > NDW ? NW - NDW : NW;      // waves with off-diagonal tiles
  static_assert(NW == NJT && NVX % 64 == 0, "one wave per 16-wide tile, whole waves of row vectors");

  int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int g = lane >> 4, c = lane & 15;
  // opaque copies of the lane coordinates: addresses derived from them are
  // recomputed in every step instead of being kept live across steps and blocks
#define CARVE_REC_FRESH() asm volatile("" : "+v"(tid), "+v"(g), "+v"(c) : : "memory")
  const int H = a.H, Tn = a.T, L = a.L, R = a.R;
  const int nbh = a.B * H, nch = Tn / L, mpc = L / W;
  const int nitems = nbh * nch;

  constexpr RecLds lay = rec_lds<T, D, RP, VAR, NB>();
  T* sU = reinterpret_cast<T*>(smem + lay.U);
  T* sX = reinterpret_cast<T*>(smem + lay.X);
  T* sV = sX;                                                 // [W] rows of v
  T* sWx = sX + lds_round(image_bytes<T, D>(W)) / sizeof(T);  // [W] rows of wx
  T* sKt = reinterpret_cast<T*>(smem + lay.Kt);
  T* sQt = reinterpret_cast<T*>(smem + lay.Qt);
  T* sKi = reinterpret_cast<T*>(smem + lay.Ki);
  T* sF = reinterpret_cast<T*>(smem + lay.F);
  T* sTau = reinterpret_cast<T*>(smem + lay.Tau);
  T* sC = reinterpret_cast<T*>(smem + lay.C);
  float* sGam = reinterpret_cast<float*>(smem + lay.Gam);     // [NB][D]
  int* sFlag = reinterpret_cast<int*>(smem + lay.Flag);
  float* sBeta = reinterpret_cast<float*>(smem + lay.Beta);
  float* sWs = sBeta + W;

  const ChunkRec cr = chunk_rec<T, D>(L, RF, NB);
  const int rs = H * D;

#define CARVE_FI() Qd::cvt(f32x4{4 * g == c ? 1.0f : 0.0f, 4 * g + 1 == c ? 1.0f : 0.0f, \
                                 4 * g + 2 == c ? 1.0f : 0.0f, 4 * g + 3 == c ? 1.0f : 0.0f})

  // ---- prefetch registers: the next block's token rows and gates ---------------
  u32x4_t cq[NXV], ck[NXV], cbx[NXV], cv[NXV], cwx[NXV];
  f32x4 pg[NB];     // g per tile (ungated)
  quad pf[NB];      // f per tile (GATED)
  f32x4 pA = zero4(), pTf = zero4();   // A, tau_f of the wave's keys 16 w + 4 g + e (GATED)
  T pbeta = (T)0.0f, pws = (T)0.0f;
  f32x4 St[NJT];    // S[v = 16 w + c][j = 16 jt + 4 g + i]
  // sources of block (BH_, first token T0_)
#define CARVE_REC_ROWS(DST_, SRC_, BH_, T0_)                                                       \
  do {                                                                                             \
    const T* s_ = reinterpret_cast<const T*>(SRC_) + ((size_t)((BH_) / H) * Tn * H + (BH_) % H) * D; \
    for (int u_ = 0; u_ < NXV; ++u_) {                                                             \
      const int x_ = tid + u_ * NT;                                                                \
      if (NVX % NT != 0 && x_ >= NVX) break;                                                       \
      (DST_)[u_] = *reinterpret_cast<const u32x4_t*>(s_ + ((T0_) + x_ / (D / VEC)) * rs + (x_ % (D / VEC)) * VEC); \
    }                                                                                              \
  } while (0)
#define CARVE_REC_PRE_KQ(BH_, T0_)                                                                 \
  do {                                                                                             \
    CARVE_REC_ROWS(cq, a.q, BH_, T0_);                                                             \
    CARVE_REC_ROWS(ck, a.k, BH_, T0_);                                                             \
    CARVE_REC_ROWS(cbx, a.bx, BH_, T0_);                                                           \
    const size_t o_ = (size_t)((BH_) / H) * Tn * H + (BH_) % H;                                    \
    if (tid < W) {                                                                                 \
      pbeta = reinterpret_cast<const T*>(a.beta)[o_ + (size_t)((T0_) + tid) * H];                  \
      if constexpr (SW) pws = reinterpret_cast<const T*>(a.wx)[o_ + (size_t)((T0_) + tid) * H];    \
    }                                                                                              \
  } while (0)
#define CARVE_REC_PRE_V(BH_, T0_)                                                                  \
  do {                                                                                             \
    CARVE_REC_ROWS(cv, a.v, BH_, T0_);                                                             \
    if constexpr (!SW) CARVE_REC_ROWS(cwx, a.wx, BH_, T0_);                                        \
  } while (0)
#define CARVE_REC_PRE_G(BH_, T0_)                                                                  \
  do {                                                                                             \
    const size_t o_ = ((size_t)((BH_) / H) * Tn * H + (BH_) % H) * D + 16 * w + 4 * g;             \
    for (int bb_ = 0; bb_ < NB; ++bb_) {                                                           \
      const size_t e_ = o_ + (size_t)(((T0_) + 16 * bb_ + c) * rs);                                \
      if constexpr (GATED) pf[bb_] = Qd::ld(reinterpret_cast<const T*>(a.f) + e_);                 \
      else pg[bb_] = *reinterpret_cast<const f32x4*>(a.g + e_);                                    \
    }                                                                                              \
    if constexpr (GATED) {                                                                         \
      pA = *reinterpret_cast<const f32x4*>(a.A + ((BH_) % H) * D + 16 * w + 4 * g);                \
      pTf = *reinterpret_cast<const f32x4*>(a.tau_f + ((BH_) % H) * D + 16 * w + 4 * g);           \
    }                                                                                              \
  } while (0)
#define CARVE_REC_PRE_S(BH_, CH_)                                                                  \
  do {                                                                                             \
    const float* s_ = a.S_chunks + ((size_t)(BH_) * nch + (CH_)) * D * D + (16 * w + c) * D + 4 * g; \
    for (int jt_ = 0; jt_ < NJT; ++jt_) St[jt_] = gload4(s_ + 16 * jt_);                           \
  } while (0)

  if (first >= nitems) return;   // (uniform over the workgroup)
  {
    const int bh = first % nbh, t0 = (nch - 1 - first / nbh) * L;
    CARVE_REC_PRE_S(bh, nch - 1 - first / nbh);
    CARVE_REC_PRE_KQ(bh, t0);
    CARVE_REC_PRE_V(bh, t0);
    CARVE_REC_PRE_G(bh, t0);
  }
  // ---- shared parameters (behind the first block's loads) -----------------------
  stage_U<T, D, RP, SW>(sU, a.Ub, a.Uw, R, tid);
  // Vb / Vw operand quads: lane (g, c) holds V[16 w + c][16 ks + 4 g + e]
  quad fVb[NRB], fVw[NRB];
  load_V<T, RP>(fVb, a.Vb, R, 16 * w + c, g);
  if constexpr (!SW) load_V<T, RP>(fVw, a.Vw, R, 16 * w + c, g);
  int* pending = nullptr;   // ready flag of the previous item, raised once its stores are complete
  int pending_val = 0;

#pragma unroll 1
  for (int item = first; item < nitems; item += stride) {
    const int row = item / nbh, bh = item % nbh, ch = nch - 1 - row;
    const int nitem = item + stride;
    const RecBuf rec(reinterpret_cast<const char*>(a.rec) + ((size_t)bh * nch + ch) * cr.total, cr.total);
    if (lead > 0 && row >= lead) {
      // follow the adjoint of this (batch, head); what the previous item still
      // has to publish goes out first
      if (pending) {
        vm_wait_all();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(pending, pending_val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        pending = nullptr;
      }
      if (tid == 0) {
        const int* p = sync + sync_adjoint_pos(nbh, nch) + bh;
        int go = 0;
        for (int n = 0; n < kLeadSpinLimit; ++n) {
          const int v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          go = v > 1 + row - lead;
          if (go || (v == 0 && n >= kPresentSpinLimit)) break;
          __builtin_amdgcn_s_sleep(4);
        }
        sFlag[15] = go;
      }
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sFlag[15]) == 0) lead = 0;
    }
    int wide_bits = 0;
#pragma unroll 1
    for (int m = 0; m < mpc; ++m) {
      // the block after this one: the chunk's next, or the next item's first
      const bool last = m + 1 == mpc;
      const bool more = !last || nitem < nitems;
      const int nbh_i = last ? nitem % nbh : bh;
      const int nch_i = last ? nch - 1 - nitem / nbh : ch;
      const int nt0 = last ? nch_i * L : ch * L + (m + 1) * W;

      // ---- R0: stage q, k, bx, beta; chunk start state ----------------------------
      CARVE_REC_FRESH();
      vm_wait_all();
      if (m == 0)
        for (int jt = 0; jt < NJT; ++jt) Qd::st(sX + RT::at(16 * w + c, 16 * jt, 4 * g), Qd::cvt(St[jt]));
      for (int u = 0; u < NXV; ++u) {
        const int x = tid + u * NT;
        if (NVX % NT != 0 && x >= NVX) break;
        stage_vec<T, D, ACT, false>(sQt, x, cq[u]);
        stage_vec<T, D, ACT, false>(sKi, x, ck[u]);
        stage_vec<T, D, false, false>(sKt, x, cbx[u]);
      }
      if (tid < W) {
        sBeta[tid] = (float)pbeta;
        rec.st(cr.Beta + 4 * m * W, 4 * tid, (float)pbeta);
        if constexpr (SW) {
          const float ws = sigmoid_f((float)pws);
          sWs[tid] = ws;
          rec.st(cr.Beta + 4 * (m * W + L), 4 * tid, ws);
        }
      }
      __syncthreads();
      if (pending) {
        if (tid == 0) __hip_atomic_store(pending, pending_val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        pending = nullptr;
      }

      // ---- R1: fold F^T[j][r] = sum_v S_hat[v][j] U[r][v] (key tile w) -------------
      CARVE_REC_FRESH();
      if (m == 0) {
        f32x4 acc[NRT];
        for (int rt = 0; rt < NRT; ++rt) acc[rt] = zero4();
        for (int vp = 0; vp < D / 32; ++vp) {
          const quad a0 = RT::tr(sX, 32 * vp, 16 * w, g, c);
          const quad a1 = RT::tr(sX, 32 * vp + 16, 16 * w, g, c);
          for (int rt = 0; rt < NRT; ++rt)
            acc[rt] = Qd::mma32(a0, a1, Qd::ld(sU + RT::at(16 * rt + c, 32 * vp, 4 * g)),
                                Qd::ld(sU + RT::at(16 * rt + c, 32 * vp + 16, 4 * g)), acc[rt]);
        }
        for (int rt = 0; rt < NRT; ++rt) {
          const quad fq = Qd::cvt(acc[rt]);
          Qd::st(sF + RT::at(16 * rt + c, 16 * w, 4 * g), fq);
          rec.st(cr.FT + rt * NT * QB, tid * QB, Qd::cvt(Qd::mma16(fq, CARVE_FI(), zero4())));
        }
        __syncthreads();
      }
      // rows of v and wx over the start state's copy (the fold is done with it)
      for (int u = 0; u < NXV; ++u) {
        const int x = tid + u * NT;
        if (NVX % NT != 0 && x >= NVX) break;
        stage_vec<T, D, false, ACT>(sV, x, cv[u]);
        if constexpr (!SW) stage_vec<T, D, false, false>(sWx, x, cwx[u]);
      }

      // ---- R2: tau^T[r][t] = tanh(F[r] . q_t) -> sTau[t][r]; q in thread order -------
      CARVE_REC_FRESH();
      for (int x = w; x < NRT * NB; x += NW) {
        const int rt = x % NRT, bb = x / NRT;
        f32x4 acc = zero4();
        for (int jp = 0; jp < D / 32; ++jp)
          acc = Qd::mma32(Qd::ld(sF + RT::at(16 * rt + c, 32 * jp, 4 * g)), Qd::ld(sF + RT::at(16 * rt + c, 32 * jp + 16, 4 * g)),
                          Qd::ld(sQt + RT::at(16 * bb + c, 32 * jp, 4 * g)),
                          Qd::ld(sQt + RT::at(16 * bb + c, 32 * jp + 16, 4 * g)), acc);
        for (int i = 0; i < 4; ++i) acc[i] = tanh_f(acc[i]);
        const quad tq = Qd::cvt(acc);
        Qd::st(sTau + RTau::at(16 * bb + c, 16 * rt, 4 * g), tq);
        rec.st(cr.Tau + ((m * W + 16 * bb) * RF + 16 * rt) * sizeof(T), (c * RF + 4 * g) * sizeof(T), tq);
      }
      for (int bb = 0; bb < NB; ++bb)
        rec.st(cr.Q + (m * NB + bb) * NT * QB, tid * QB, RT::tr(sQt, 16 * bb, 16 * w, g, c));
      __syncthreads();

      // ---- R3: gates (log retentions in units of log 2) ------------------------------
      CARVE_REC_FRESH();
      // key side, key tile w: lane (g, c) of tile bb holds t = 16 bb + c and
      // j = 16 w + 4 g + i; the prefix sums run along the 16 lanes of a row
      f32x4 lam[NB];
      {
        f32x4 carry = zero4();
        f32x4 na = zero4(), tf = zero4();
        if constexpr (GATED) {
          for (int i = 0; i < 4; ++i) na[i] = -expf(pA[i]);
          tf = pTf;
        }
        for (int bb = 0; bb < NB; ++bb) {
          f32x4 z = zero4();
          for (int ks = 0; ks < NRB; ++ks)
            z = Qd::mma16(fVb[ks], Qd::ld(sTau + RTau::at(16 * bb + c, 16 * ks, 4 * g)), z);
          const f32x4 bxv = Qd::f32(Qd::ld(sKt + RT::at(16 * bb + c, 16 * w, 4 * g)));
          f32x4 gv, sgv;
          if constexpr (GATED) {
            const f32x4 fv = Qd::f32(pf[bb]);
            for (int i = 0; i < 4; ++i) gv[i] = na[i] * softplus2_f(fv[i] + tf[i]);   // g / log 2
          } else {
            gv = pg[bb];
          }
          for (int i = 0; i < 4; ++i) {
            const float zz = z[i] + bxv[i];
            const float ex = exp2_f(-fabsf(zz) * kLog2e);
            const float rc = fast_rcp(1.0f + ex);
            const float sp = fmaf(fmaxf(zz, 0.0f), kLog2e, __builtin_amdgcn_logf(1.0f + ex));
            sgv[i] = zz >= 0.0f ? rc : ex * rc;
            const float ell = GATED ? gv[i] - sp : fmaf(gv[i], kLog2e, -sp);
            lam[bb][i] = bb == 0 ? row_scan(ell) : carry[i] + row_scan(ell);
            carry[i] = row_bcast15(lam[bb][i]);
          }
          rec.st(cr.Sig + (m * NB + bb) * NT * QB, tid * QB, Qd::cvt(sgv));
        }
      }
      bool wide = false;
      if constexpr (NB > 1) {
        bool mine = false;
        for (int i = 0; i < 4; ++i) mine = mine || row_bcast15(lam[NB - 1][i]) < -kBwdWideLog * kLog2e;
        const bool wv_wide = __any(mine) != 0;
        if (lane == 0) sFlag[w] = wv_wide ? 1 : 0;
      }
      // value side, value tile w: rows t = 16 bb + 4 g + i, column v = 16 w + c
      f32x4 wv[NB];
      for (int bb = 0; bb < NB; ++bb) {
        const quad vq = RT::tr(sV, 16 * bb, 16 * w, g, c);
        rec.st(cr.V + (m * NB + bb) * NT * QB, tid * QB, vq);
        const f32x4 vv = Qd::f32(vq);
        if constexpr (SW) {
          wv[bb] = *reinterpret_cast<const f32x4*>(sWs + 16 * bb + 4 * g) * vv;
        } else {
          f32x4 z = Qd::f32(RT::tr(sWx, 16 * bb, 16 * w, g, c));
          for (int ks = 0; ks < NRB; ++ks)
            z = Qd::mma16(Qd::ld(sTau + RTau::at(16 * bb + c, RP + 16 * ks, 4 * g)), fVw[ks], z);
          for (int i = 0; i < 4; ++i) z[i] = sigmoid_f(z[i]);
          rec.st(cr.W + (m * NB + bb) * NT * 16, tid * 16, z);
          wv[bb] = z * vv;
        }
        wv[bb] *= *reinterpret_cast<const f32x4*>(sBeta + 16 * bb + 4 * g);   // beta w v
      }
      __syncthreads();
      if constexpr (NB > 1) {
        int f = 0;
        for (int x = 0; x < NW; ++x) f |= sFlag[x];
        wide = __builtin_amdgcn_readfirstlane(f) != 0;
        if (wide) wide_bits |= 1 << m;
      }
      // decayed operands of the key tile, in place of the raw rows
      {
        f32x4 fill, cprev = zero4();
        for (int i = 0; i < 4; ++i) fill[i] = exp2_f(-0.5f * row_bcast15(lam[NB - 1][i]));   // e^{-rho}
        for (int bb = 0; bb < NB; ++bb) {
          const int ro = RT::at(16 * bb + c, 16 * w, 4 * g);
          const f32x4 kv = Qd::f32(Qd::ld(sKi + ro)), qv = Qd::f32(Qd::ld(sQt + ro));
          const float bt = sBeta[16 * bb + c];
          f32x4 kt, qt, ki, ev, gm;
          for (int i = 0; i < 4; ++i) {
            float rho = 0.5f * row_bcast15(lam[NB - 1][i]), x = lam[bb][i];
            if (NB > 1 && wide) {
              // tile by tile: relative to the tile's start and middle
              const float ce = row_bcast15(lam[bb][i]);
              x -= cprev[i];
              rho = 0.5f * (ce - cprev[i]);
              fill[i] = exp2_f(-rho);
              cprev[i] = ce;
            }
            float E, Ei;
            exp2_pm(x - rho, E, Ei);
            kt[i] = bt * (kv[i] * row_shr1(E, fill[i]));
            qt[i] = qv[i] * E;
            ki[i] = kv[i] * Ei;
            ev[i] = E;
            gm[i] = exp2_f(rho);
            fill[i] = row_bcast15(E);   // one reference: E of the tile's last token
          }
          Qd::st(sKt + ro, Qd::cvt(kt));
          Qd::st(sQt + ro, Qd::cvt(qt));
          Qd::st(sKi + ro, Qd::cvt(ki));
          rec.st(cr.E + (m * NB + bb) * NT * 16, tid * 16, ev);
          if (c == 0 && (bb == 0 || wide)) {
            *reinterpret_cast<f32x4*>(sGam + bb * D + 16 * w + 4 * g) = gm;
            rec.st(cr.Gam + ((m * NB + bb) * D + 16 * w) * 4, 16 * g, gm);
          }
        }
      }
      if (more) CARVE_REC_PRE_KQ(nbh_i, nt0);
      __syncthreads();

      // ---- R4: S' for its transposition; diagonal inverses, coupling tiles, S' Kh ----
      CARVE_REC_FRESH();
      quad sb[NJT];   // S' of the block (or, tile by tile, of its first tile)
      for (int jt = 0; jt < NJT; ++jt) {
        sb[jt] = Qd::cvt(St[jt] * *reinterpret_cast<const f32x4*>(sGam + 16 * jt + 4 * g));
        Qd::st(sX + RT::at(16 * w + c, 16 * jt, 4 * g), sb[jt]);
      }
      if (more) CARVE_REC_PRE_V(nbh_i, nt0);
      if (w >= NW - NDW) {
        typedef Quad<float> Qf;
        for (int i = NW - 1 - w; i < NB; i += NDW) {
          f32x4 acc = zero4(), accT = zero4();
          for (int jp = 0; jp < D / 32; ++jp) {
            const int o0 = RT::at(16 * i + c, 32 * jp, 4 * g), o1 = RT::at(16 * i + c, 32 * jp + 16, 4 * g);
            const quad k0 = Qd::ld(sKt + o0), k1 = Qd::ld(sKt + o1), i0 = Qd::ld(sKi + o0), i1 = Qd::ld(sKi + o1);
            acc = Qd::mma32(k0, k1, i0, i1, acc);     // Kh_{t = 4 g + e} . Ki_{s = c}
            accT = Qd::mma32(i0, i1, k0, k1, accT);   // Ki_{s = 4 g + e} . Kh_{t = c}
          }
          T* tt = sC + (NTP + NTA + i) * ST::N;
          if constexpr (sizeof(T) == 4) {
            // f32: T[c][s] = delta(c, s) - sum_{t > s} T[c][t] A[t][s], s = 15 .. 0,
            // row c in lane c, from A^T parked in T's own place (one wave, whose
            // LDS accesses are in order).  The product form below loses T to
            // cancellation where the keys are alike: relative error 8e-5 for
            // equal keys, 6e-8 by substitution (below bf16's rounding, but not
            // below f32's).
            f32x4 av;
            for (int e = 0; e < 4; ++e) av[e] = (c < 4 * g + e) ? acc[e] : 0.0f;
            Qd::st(tt + ST::at(c, 4 * g), av);   // A[4 g + e][c] in row c
            asm volatile("" ::: "memory");
            float x[16];
#pragma unroll
            for (int s = 15; s >= 0; --s) {
              float acc0 = (s == c) ? 1.0f : 0.0f, acc1 = 0.0f;
#pragma unroll
              for (int t = s + 1; t < 16; ++t) {
                if ((t - s) & 1) acc0 -= x[t] * tt[ST::at(s, t)];
                else acc1 -= x[t] * tt[ST::at(s, t)];
              }
              x[s] = acc0 + acc1;
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (g == k) Qd::st(tt + ST::at(c, 4 * k), f32x4{x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]});
          } else {
            // T = (I + A)^{-1} = (I + M)(I + M^2)(I + M^4)(I + M^8), M = -A (M^16 = 0)
            f32x4 mB, mA, I4;   // M in the result layout (M[4g+e][c]) and transposed (M[c][4g+e])
            for (int e = 0; e < 4; ++e) {
              mB[e] = (c < 4 * g + e) ? -acc[e] : 0.0f;
              mA[e] = (4 * g + e < c) ? -accT[e] : 0.0f;
              I4[e] = (4 * g + e == c) ? 1.0f : 0.0f;
            }
            const f32x4 M2 = Qf::mma16(mA, mB, zero4());
            const f32x4 M2t = Qf::mma16(mB, mA, zero4());
            const f32x4 M4 = Qf::mma16(M2t, M2, zero4());
            const f32x4 M4t = Qf::mma16(M2, M2t, zero4());
            // the factors commute; formed transposed (rows s, columns t), so that
            // a lane's four elements are one row quad of T: T[c][4g..4g+3]
            const f32x4 M8t = Qf::mma16(M4, M4t, zero4());
            const f32x4 X1 = Qf::mma16(M4 + I4, M8t + I4, zero4());
            const f32x4 X2 = Qf::mma16(M2 + I4, X1, zero4());
            f32x4 Tt = Qf::mma16(mB + I4, X2, zero4());
            for (int e = 0; e < 4; ++e) Tt[e] = 4 * g + e < c ? Tt[e] : 0.0f;
            Qd::st(tt + ST::at(c, 4 * g), Qd::cvt(Tt));
          }
        }
      }
      if (NOW == NW || w < NOW) {
        int ct = c, gt = g;
        asm volatile("" : "+v"(ct), "+v"(gt));
#pragma unroll 1
        for (int x = w; x < NTP + NTA; x += NOW) {
          const bool isA = x >= NTP;
          const int y = isA ? x - NTP : x;
          const int i = tri_row_of(y, isA), j = tri_col_of(y, isA);
          // acc[e] = Ki_{s = 16 j + 4 g + e} . X_{t = 16 i + c}, X = Kh (A) or Qt (P)
          const T* bsrc = isA ? sKt : sQt;
          f32x4 acc = zero4();
          for (int jp = 0; jp < D / 32; ++jp)
            acc = Qd::mma32(Qd::ld(sKi + RT::at(16 * j + ct, 32 * jp, 4 * gt)), Qd::ld(sKi + RT::at(16 * j + ct, 32 * jp + 16, 4 * gt)),
                            Qd::ld(bsrc + RT::at(16 * i + ct, 32 * jp, 4 * gt)),
                            Qd::ld(bsrc + RT::at(16 * i + ct, 32 * jp + 16, 4 * gt)), acc);
          f32x4 val;
          for (int e = 0; e < 4; ++e) val[e] = isA ? -acc[e] : (i > j || 4 * gt + e <= ct) ? acc[e] : 0.0f;
          Qd::st(sC + x * ST::N + ST::at(ct, 4 * gt), Qd::cvt(val));
        }
      }
      // R = beta w v - Kh S'^T on the value tile (rows t = 16 bb + 4 g + e)
      const int nxk = wide ? 1 : NB;
      for (int bb = 0; bb < NB; ++bb) {
        if (bb < nxk) {
          f32x4 xk = zero4();
          for (int jp = 0; jp < NJT / 2; ++jp)
            xk = Qd::mma32(Qd::ld(sKt + RT::at(16 * bb + c, 32 * jp, 4 * g)), Qd::ld(sKt + RT::at(16 * bb + c, 32 * jp + 16, 4 * g)),
                           sb[2 * jp], sb[2 * jp + 1], xk);
          wv[bb] -= xk;
        }
      }
      __syncthreads();

      // ---- R5: u; records of S', K, C; state update where a block follows -----------
      CARVE_REC_FRESH();
      if (more) CARVE_REC_PRE_G(nbh_i, nt0);
      quad uq[NB];
      if (!wide) {
        for (int i = 0; i < NB; ++i) {
          f32x4 r = wv[i];
          for (int j = 0; j < i; ++j)
            r = Qd::mma16(Qd::ld(sC + (NTP + tri_strict(i, j)) * ST::N + ST::at(c, 4 * g)), uq[j], r);
          uq[i] = Qd::cvt(ST::apply_T(Qd::ld(sC + (NTP + NTA + i) * ST::N + ST::at(c, 4 * g)), r));
        }
        for (int vt = 0; vt < NJT; ++vt) rec.st(cr.S + (m * NB * NJT + vt) * NT * QB, tid * QB, RT::tr(sX, 16 * vt, 16 * w, g, c));
        if (!last) {
          // S <- (S' + u^T Ki) diag(e^{rho})
          for (int jt = 0; jt < NJT; ++jt) {
            const f32x4 er = *reinterpret_cast<const f32x4*>(sGam + 16 * jt + 4 * g);
            f32x4 acc = St[jt] * er;
            for (int bb = 0; bb < NB; ++bb) acc = Qd::mma16(RT::tr(sKi, 16 * bb, 16 * jt, g, c), uq[bb], acc);
            St[jt] = acc * er;
          }
        }
      } else {
        // tile by tile: the state runs through the block
        for (int bb = 0; bb < NB; ++bb) {
          if (bb > 0) {
            for (int jt = 0; jt < NJT; ++jt) {
              sb[jt] = Qd::cvt(St[jt] * *reinterpret_cast<const f32x4*>(sGam + bb * D + 16 * jt + 4 * g));
              Qd::st(sX + RT::at(16 * w + c, 16 * jt, 4 * g), sb[jt]);
            }
            f32x4 xk = zero4();
            for (int jp = 0; jp < NJT / 2; ++jp)
              xk = Qd::mma32(Qd::ld(sKt + RT::at(16 * bb + c, 32 * jp, 4 * g)), Qd::ld(sKt + RT::at(16 * bb + c, 32 * jp + 16, 4 * g)),
                             sb[2 * jp], sb[2 * jp + 1], xk);
            wv[bb] -= xk;
            __syncthreads();
          }
          uq[bb] = Qd::cvt(ST::apply_T(Qd::ld(sC + (NTP + NTA + bb) * ST::N + ST::at(c, 4 * g)), wv[bb]));
          for (int vt = 0; vt < NJT; ++vt) rec.st(cr.S + ((m * NB + bb) * NJT + vt) * NT * QB, tid * QB, RT::tr(sX, 16 * vt, 16 * w, g, c));
          for (int jt = 0; jt < NJT; ++jt) {
            const f32x4 er = *reinterpret_cast<const f32x4*>(sGam + bb * D + 16 * jt + 4 * g);
            St[jt] = Qd::mma16(RT::tr(sKi, 16 * bb, 16 * jt, g, c), uq[bb], St[jt] * er) * er;
          }
          if (bb + 1 < NB) __syncthreads();   // the next tile's S' replaces this one's
        }
      }
      if (last && more) CARVE_REC_PRE_S(nbh_i, nch_i);
      CARVE_REC_FRESH();
      // u as rows of tokens, straight into its tile image
      for (int bb = 0; bb < NB; ++bb)
        rec.st(cr.U + image_bytes<T, D>(W) * m + 16 * bb * RT::LD * sizeof(T), RT::at(c, 16 * w, 4 * g) * sizeof(T),
               Qd::cvt(Qd::mma16(uq[bb], CARVE_FI(), zero4())));
      {
        // tile images of Kh, Qt, Ki (consecutive in LDS) and of the coupling tiles
        constexpr int NVK = (int)(image_bytes<T, D>(W) / 16);
        static_assert(image_bytes<T, D>(W) % 16 == 0 && ctile_bytes<T>(NB) % 16 == 0, "whole 16-byte vectors");
        const u32x4_t* sk = reinterpret_cast<const u32x4_t*>(smem + lay.Kt);
        for (int x = tid; x < 3 * NVK; x += NT) rec.st(cr.K + 3 * image_bytes<T, D>(W) * m, x * 16, sk[x]);
        constexpr int NVC = (int)(ctile_bytes<T>(NB) / 16);
        const u32x4_t* sc = reinterpret_cast<const u32x4_t*>(smem + lay.C);
        for (int x = tid; x < NVC; x += NT) rec.st(cr.C + ctile_bytes<T>(NB) * m, x * 16, sc[x]);
      }
      __syncthreads();
    }  // blocks of the chunk
    pending = sync + (size_t)bh * nch + ch;
    pending_val = 1 | (wide_bits << 1);
  }  // items
  // the last item's flag
  vm_wait_all();
  __syncthreads();
  if (tid == 0 && pending) __hip_atomic_store(pending, pending_val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#undef CARVE_REC_FRESH
#undef CARVE_REC_ROWS
#undef CARVE_REC_PRE_KQ
#undef CARVE_REC_PRE_V
#undef CARVE_REC_PRE_G
#undef CARVE_REC_PRE_S
#undef CARVE_FI
}

}  // namespace carve

// carve_dev.h -- device-side building blocks shared by the CARVE kernels
// (gfx950 / CDNA4, wave64).
//
// Matrix-core tiles.  Every product in the layer is a 16x16 output tile on the
// matrix cores (Quad below), with f32 accumulation:
//   bf16 operands: v_mfma_f32_16x16x32_bf16 and v_mfma_f32_16x16x16_bf16
//   f32  operands: v_mfma_f32_16x16x4_f32, eight or four for the same depth
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

namespace carve {

// ---- K16 "quad" operands --------------------------------------------------
// The kernels issue their products on K16 (and paired K32) matrix-core steps.
// For one 16x16 output tile and one 16-wide slice of the contraction index k:
//   lane l = 16 g + c supplies A[m = c][k = 4g .. 4g+3]  and  B[k = 4g .. 4g+3][n = c]
//   and receives C[m = 4g + i][n = c], i = 0..3.
// So an accumulator tile X held in registers is directly a B operand whose K is
// X's row index, and an A operand representing X^T.  LDS operands are read as
// 4-element quads either along a row ("natural": lane c reads row c) or across
// four rows ("transposed": lane c reads column c), the latter with the gfx950
// transposing LDS read for 16-bit data.
//
// One accumulator takes either K16 or K32 steps: a bf16 mma16 directly on the
// result of a mma32, or the other way round, gets no wait states from the
// compiler and the card then returns wrong values (K16 on K32: rows 0 and 1 of
// every quad, K32 on K16: rows 2 and 3; measured, every time).  Chains of both
// kinds are added at the end, or lie a barrier apart; tests/test_mfma_hazards.py
// checks the distances in the compiled library.
template <typename T>
struct Quad;

template <>
struct Quad<bf16_t> {
  typedef bf16x4 q;
  static __device__ __forceinline__ q ld(const bf16_t* p) { return *reinterpret_cast<const bf16x4*>(p); }
  // lane (g, c) receives buf[r0 + 4g + e][c0 + c], e = 0..3
  static __device__ __forceinline__ q ld_tr(const bf16_t* buf, int ld, int r0, int c0, int g, int c) {
    typedef short short4_ __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4_ lds_s4;
    const bf16_t* p = buf + (r0 + 4 * g + (c >> 2)) * ld + c0 + 4 * (c & 3);
    const short4_ v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p));
    return __builtin_bit_cast(bf16x4, v);
  }
  // ld_tr on a quad-swizzled tile (qswz below); r0 a multiple of 16, so the
  // swizzle term of every row this lane touches is g
  static __device__ __forceinline__ q ld_tr_sw(const bf16_t* buf, int ld, int r0, int c0, int g, int c) {
    return ld_tr_at(buf + (r0 + 4 * g + (c >> 2)) * ld + c0 + 4 * ((c & 3) ^ g));
  }
  // transposing read with the lane's own address (lane (g, c) names row
  // r0 + 4 g + c / 4, quad c % 4 of the 16 columns)
  static __device__ __forceinline__ q ld_tr_at(const bf16_t* p) {
    typedef short short4_ __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4_ lds_s4;
    const short4_ v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p));
    return __builtin_bit_cast(bf16x4, v);
  }
  static __device__ __forceinline__ void st(bf16_t* p, q v) { *reinterpret_cast<bf16x4*>(p) = v; }
  static __device__ __forceinline__ q cvt(f32x4 x) {
    // by pairs, one conversion instruction each: from a four-element conversion
    // the compiler converts every value on its own and packs them afterwards
    const f32x2 a = {x[0], x[1]}, b = {x[2], x[3]};
    const u32x2_t r = {__builtin_bit_cast(unsigned, __builtin_convertvector(a, bf16x2)),
                       __builtin_bit_cast(unsigned, __builtin_convertvector(b, bf16x2))};
    return __builtin_bit_cast(q, r);
  }
  static __device__ __forceinline__ f32x4 f32(q x) {
    f32x4 o = {(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
    return o;
  }
  static __device__ __forceinline__ f32x4 mma16(q a, q b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
  }
  // two K16 slices in one K32 step (the same slice pairing on both sides)
  static __device__ __forceinline__ f32x4 mma32(q a0, q a1, q b0, q b1, f32x4 c) {
    const bf16x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    const bf16x8 b = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Quad<float> {
  typedef f32x4 q;
  static __device__ __forceinline__ q ld(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
  static __device__ __forceinline__ q ld_tr(const float* buf, int ld, int r0, int c0, int g, int c) {
    const float* p = buf + (r0 + 4 * g) * ld + c0 + c;
    q o = {p[0], p[ld], p[2 * ld], p[3 * ld]};
    return o;
  }
  // f32 tiles are not swizzled (qswz<float> is 0)
  static __device__ __forceinline__ q ld_tr_sw(const float* buf, int ld, int r0, int c0, int g, int c) {
    return ld_tr(buf, ld, r0, c0, g, c);
  }
  static __device__ __forceinline__ void st(float* p, q v) { *reinterpret_cast<f32x4*>(p) = v; }
  static __device__ __forceinline__ q cvt(f32x4 x) { return x; }
  static __device__ __forceinline__ f32x4 f32(q x) { return x; }
  static __device__ __forceinline__ f32x4 mma16(q a, q b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], c, 0, 0, 0);
    return c;
  }
  static __device__ __forceinline__ f32x4 mma32(q a0, q a1, q b0, q b1, f32x4 c) {
    return mma16(a1, b1, mma16(a0, b0, c));
  }
};

// ---- bank-conflict-free bf16 operand tiles -----------------------------------
// The LDS serves 8-byte lane accesses in groups: reads (row-wise or
// transposing) 32 lanes at a time against a 256-byte bank window, writes 16
// lanes at a time against a 128-byte window.  A row-major bf16 tile is read and
// written in three quad (8-byte) patterns: 16 rows x 2 quads (row-wise read),
// 8 rows x 4 quads (transposing read) and 16 rows x 1 quad (write of a result
// tile).  Row padding alone cannot make all three conflict-free.  With a row
// stride of x quads, x = 4 (mod 8), and quad q of row r stored at quad
// q ^ ((r >> 2) & 3), all three are: the XOR spreads the rows that the stride
// maps to one window position.  The term only touches the quad index's two low
// bits, so offsets along a row stay additive.
// qswz<T>(r): the element-index XOR of row r (f32 tiles: none).
template <typename T>
__device__ __forceinline__ int qswz(int r) {
  return sizeof(T) == 2 ? ((r >> 2) & 3) << 2 : 0;
}

// global 4-element vector of the token dtype <-> f32x4
__device__ __forceinline__ f32x4 gload4(const bf16_t* p) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  f32x4 o = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
  return o;
}
__device__ __forceinline__ f32x4 gload4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// Row and column of tile y of a row-major enumeration of the lower-triangular
// 16-token tiles of a block of up to four: inclusive (j <= i) or strict (j < i).
// From packed digits: the tile loops are short and wave-uniform, and counting
// rows with compares and branches took as long as the tile's products.
__device__ __forceinline__ int tri_row_of(int y, bool strict) {
  return (int)((strict ? 0x333221ull : 0x3333222110ull) >> (4 * y)) & 15;
}
__device__ __forceinline__ int tri_col_of(int y, bool strict) {
  return (int)((strict ? 0x210100ull : 0x3210210100ull) >> (4 * y)) & 15;
}

// Chunk-record accesses between compute units of different XCDs: buffer
// operations at agent scope (sc1).  Such a store goes through the XCD's L2 to
// the coherence point, and such a load comes from there, so that publishing a
// record needs no write-back of the whole L2 and reading it no invalidation:
// a wait for the writer's stores and a flag are enough.  The address is a
// uniform base (the record), a uniform byte offset and a 32-bit lane offset.
typedef unsigned u32x4_g __attribute__((ext_vector_type(4)));
struct RecBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ RecBuf(const void* base, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00027000)) {}
  static constexpr int kAgent = 16;   // sc1
  template <typename V>
  __device__ __forceinline__ void st(unsigned off, unsigned lane_off, V v) const {
    // 16 bytes: the whole offset in the vector operand.  With part of it in a
    // scalar register the compiler takes the store data as read at issue and
    // lets the next instruction overwrite a data register; under contention for the
    // memory path the last lanes then stored the new value (seen in the erase
    // gate of f32 layers with more than 512 workgroups on the card).
    if constexpr (sizeof(V) == 16)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_g, v), r, (int)(off + lane_off), 0, kAgent);
    else if constexpr (sizeof(V) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, (int)lane_off, (int)off, kAgent);
    else
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)lane_off, (int)off, kAgent);
  }
  template <typename V>
  __device__ __forceinline__ V ld(unsigned off, unsigned lane_off) const {
    if constexpr (sizeof(V) == 16)
      return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, kAgent));
    else if constexpr (sizeof(V) == 8)
      return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, kAgent));
    else
      return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)off, kAgent));
  }
};

// DPP helpers inside rows of 16 lanes
// x of the lane one to the left in its row; the first lane of a row gets fill
__device__ __forceinline__ float row_shr1(float x, float fill) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, fill), __builtin_bit_cast(int, x),
                                                               0x111, 0xf, 0xf, false));
}
// x of the lane one to the right in its row; the last lane of a row gets fill
__device__ __forceinline__ float row_shl1(float x, float fill) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, fill), __builtin_bit_cast(int, x),
                                                               0x101, 0xf, 0xf, false));
}
// x of lane 15 of the row, in every lane of the row (every lane is written, so
// no old value is needed)
__device__ __forceinline__ float row_bcast15(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x15F, 0xf, 0xf, false));
}
// x of lane 0 of the row, in every lane of the row
__device__ __forceinline__ float row_bcast0(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150, 0xf, 0xf, false));
}
// x of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ float lane_xor1(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));
}
// wait until every vector memory operation this wave issued has completed
__device__ __forceinline__ void vm_wait_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// inclusive suffix sum over the 16 lanes of each row
__device__ __forceinline__ float row_suffix(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x101, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x102, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x104, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x108, 0xf, 0xf, false));
  return x;
}
// inclusive prefix sum over the 16 lanes of each row
__device__ __forceinline__ float row_scan(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x111, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x112, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x114, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x118, 0xf, 0xf, false));
  return x;
}

__device__ __forceinline__ f32x4 zero4() {
  f32x4 z = {0.f, 0.f, 0.f, 0.f};
  return z;
}

// ---- elementwise math (f32, hardware exp2/log2/rcp) -----------------------
__device__ __forceinline__ float fast_exp(float x) { return __expf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float sigmoid_f(float z) { return fast_rcp(1.0f + fast_exp(-z)); }
// base-2 forms for code that keeps log retentions in units of log 2 (every
// exponential then is one hardware exp2, with no scaling product)
constexpr float kLog2e = 1.44269504088896341f;
__device__ __forceinline__ float exp2_f(float y) { return __builtin_amdgcn_exp2f(y); }
// 2^y and 2^-y
__device__ __forceinline__ void exp2_pm(float y, float& ep, float& em) {
  ep = __builtin_amdgcn_exp2f(y);
  em = __builtin_amdgcn_exp2f(-y);
}
// softplus(z) / log 2 = log2(1 + e^z) without overflow (the log2 argument is
// in [1, 2])
__device__ __forceinline__ float softplus2_f(float z) {
  return fmaf(fmaxf(z, 0.0f), kLog2e, __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-fabsf(z) * kLog2e)));
}
// natural log of x in [1, 2]: the hardware log2 and one product (no range
// reduction or denormal scaling is needed there)
__device__ __forceinline__ float log_1to2(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945f; }
// softplus(z) = log(1 + e^z) and sigmoid(z) from one exponential
__device__ __forceinline__ void softplus_sigmoid(float z, float& sp, float& sig) {
  const float e = fast_exp(-fabsf(z));
  const float r = fast_rcp(1.0f + e);
  sp = fmaxf(z, 0.0f) + log_1to2(1.0f + e);
  sig = z >= 0.0f ? r : e * r;
}
// tanh with a short odd series near 0 (the exp form cancels there)
__device__ __forceinline__ float tanh_f(float y) {
  const float big = 1.0f - 2.0f * fast_rcp(fast_exp(2.0f * y) + 1.0f);
  const float y2 = y * y;
  const float small = y * (1.0f + y2 * (-1.0f / 3.0f + y2 * (2.0f / 15.0f + y2 * (-17.0f / 315.0f))));
  return fabsf(y) < 0.125f ? small : big;
}

// ---- input activations (queries and keys: SiLU then L2 norm; values: SiLU) --
__device__ __forceinline__ float silu_f(float x) { return x * sigmoid_f(x); }
// d SiLU / dx = sigmoid(x) (1 + x (1 - sigmoid(x)))
__device__ __forceinline__ float silu_grad_f(float x) {
  const float s = sigmoid_f(x);
  return s * (1.0f + x * (1.0f - s));
}
__device__ __forceinline__ f32x4 silu4(f32x4 x) {
  f32x4 o;
  for (int e = 0; e < 4; ++e) o[e] = silu_f(x[e]);
  return o;
}
__device__ __forceinline__ f32x4 silu_grad4(f32x4 x) {
  f32x4 o;
  for (int e = 0; e < 4; ++e) o[e] = silu_grad_f(x[e]);
  return o;
}
// the L2 normalisation is x / sqrt(|x|^2 + eps)
constexpr float kL2Eps = 1e-6f;

// sum over aligned groups of N consecutive lanes (N a power of two dividing
// 64), in every lane of the group; every lane of the wave must take part.
// Within a row of 16 lanes a DPP butterfly (lane ^ 1, lane ^ 2, then the
// half-row and row mirrors, which pair each lane with one in the other half);
// across rows lane shuffles.  Every step adds two values in either order, so
// all lanes of a group get the bitwise same sum.
template <int N>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(N >= 1 && N <= 64 && (N & (N - 1)) == 0, "power of two up to a wave");
  if constexpr (N >= 2)
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));
  if constexpr (N >= 4)
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x4E, 0xf, 0xf, false));
  if constexpr (N >= 8)   // row_half_mirror: lane i <-> 7 - i within each half-row
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x141, 0xf, 0xf, false));
  if constexpr (N >= 16)  // row_mirror: lane i <-> 15 - i within each row
    x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x140, 0xf, 0xf, false));
  if constexpr (N >= 32) x += __shfl_xor(x, 16);
  if constexpr (N >= 64) x += __shfl_xor(x, 32);
  return x;
}

// 16 bytes of the token dtype <-> floats
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
template <typename T>
struct Chunk16;
template <>
struct Chunk16<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(u32x4_t v, float* f) {
    const bf16x8 b = __builtin_bit_cast(bf16x8, v);
    for (int i = 0; i < 8; ++i) f[i] = (float)b[i];
  }
  static __device__ __forceinline__ u32x4_t pack(const float* f) {
    bf16x8 b;
    for (int i = 0; i < 8; ++i) b[i] = (bf16_t)f[i];
    return __builtin_bit_cast(u32x4_t, b);
  }
};
template <>
struct Chunk16<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(u32x4_t v, float* f) {
    const f32x4 b = __builtin_bit_cast(f32x4, v);
    for (int i = 0; i < 4; ++i) f[i] = b[i];
  }
  static __device__ __forceinline__ u32x4_t pack(const float* f) {
    const f32x4 b = {f[0], f[1], f[2], f[3]};
    return __builtin_bit_cast(u32x4_t, b);
  }
};

// Sum over a row of SiLU(raw)^2, the row spread as 16-byte chunks over NC
// consecutive lanes (every lane of the wave must take part); returns
// 1 / sqrt(sum + eps), in every lane of the row.
template <typename T, int NC>
__device__ __forceinline__ float act_row_inv_norm(u32x4_t raw) {
  float f[Chunk16<T>::N];
  Chunk16<T>::unpack(raw, f);
  float ss = 0.0f;
  for (int i = 0; i < Chunk16<T>::N; ++i) {
    const float sv = silu_f(f[i]);
    ss += sv * sv;
  }
  return rsqrtf(group_sum<NC>(ss) + kL2Eps);
}
// SiLU(raw) * scale of one chunk
template <typename T>
__device__ __forceinline__ u32x4_t act_chunk(u32x4_t raw, float scale) {
  float f[Chunk16<T>::N];
  Chunk16<T>::unpack(raw, f);
  for (int i = 0; i < Chunk16<T>::N; ++i) f[i] = silu_f(f[i]) * scale;
  return Chunk16<T>::pack(f);
}

}  // namespace carve

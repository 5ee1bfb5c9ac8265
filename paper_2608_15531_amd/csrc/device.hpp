// Device helpers shared by the fused, unfused and decode kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace fqk {

typedef __bf16 bf16x8_t __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef __bf16 bf16x2_t __attribute__((__vector_size__(2 * sizeof(__bf16))));
typedef float f32x4_t __attribute__((__vector_size__(4 * sizeof(float))));
typedef uint32_t u32x4_t __attribute__((__vector_size__(4 * sizeof(uint32_t))));

// ---------------------------------------------------------------------------
// INT4 -> bf16 MFMA operand.
//
// A 32-bit word of Wq holds the codes of 8 consecutive k of one column, code
// j in bits 4j..4j+3.  The bf16 value 128 + q has bit pattern 0x4300 | q
// (exponent 2^7, q in the low four mantissa bits, whose unit is 1), so one
// and-or turns the codes sitting in bits 0..3 and 16..19 of a word into a
// packed bf16 pair without any conversion instruction: the pairs come out as
// (k0,k4), (k1,k5), (k2,k6), (k3,k7) after shifts by 0, 4, 8 and 12.  The
// activation operand is staged in that same order, so the 8-term dot product
// the MFMA forms per lane is unchanged.  The offset 128 + z is removed after
// each 128-row group with the exact identity
//     sum_k x_k (q_k - z) = sum_k x_k (128 + q_k) - (128 + z) sum_k x_k,
// so (q - z) never needs to be formed and the scale s is applied in fp32 once
// per group (eq. 3 of the paper).  The fp32 sums are at most 143 sum|x_k|,
// which keeps their rounding error near 1e-6 of the result.
// ---------------------------------------------------------------------------
// (a & b) | c as one VALU operation (gfx950 three-input bitwise op; truth
// table 0xEA).  Plain C++ for this pattern compiles to two VOP2 operations,
// because a VOP3 encoding cannot carry the two literal constants.
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xEA);
}

constexpr float kCodeOffset = 128.f;   // value of the bf16 bit pattern 0x4300

// Two words (two columns) at once, each into its 8-element operand: the
// and-or above on the word shifted by 0, 4, 8 and 12.  One 64-bit shift of
// the pair (w1:w0) yields w1 >> s in its high half and w0 >> s in its low
// half, polluted only in bits 32-s..31 by w1's low bits, which the nibble mask
// clears for s <= 12, so three 64-bit shifts replace six 32-bit ones.
template <int S>
__device__ __forceinline__ uint64_t shr64c(uint64_t p) {
  uint64_t r;
  asm("v_lshrrev_b64 %0, %2, %1" : "=v"(r) : "v"(p), "i"(S));
  return r;
}

// VM holds the mask and the bias in vector registers, otherwise the compiler
// keeps them in scalar ones.  It gains where every code word meets 64 rows
// (row-block kernel, 4096 x 28672 at 128 rows 67.0 -> 65.9 us, 4096 x 6144 21.5 ->
// 21.2) and costs the strip kernel's two-block waves (14336 x 4096 at 27 rows 18.8
// -> 19.1, 4096 x 14336 at 32 rows 16.8 -> 16.9); at up to 16 rows it changes
// nothing.
template <bool VM>
__device__ __forceinline__ void dequant_pair(uint32_t w0, uint32_t w1, bf16x8_t& b0, bf16x8_t& b1) {
  uint32_t mask = 0x000F000Fu, bias = 0x43004300u;
  if constexpr (VM) {
    asm("v_mov_b32 %0, 0x000f000f" : "=v"(mask));
    asm("v_mov_b32 %0, 0x43004300" : "=v"(bias));
  }
  const uint64_t p = (uint64_t(w1) << 32) | w0;
  const uint64_t s4 = shr64c<4>(p), s8 = shr64c<8>(p), s12 = shr64c<12>(p);
  u32x4_t r0, r1;
  r0[0] = and_or(w0, mask, bias);
  r1[0] = and_or(w1, mask, bias);
  r0[1] = and_or(uint32_t(s4), mask, bias);
  r1[1] = and_or(uint32_t(s4 >> 32), mask, bias);
  r0[2] = and_or(uint32_t(s8), mask, bias);
  r1[2] = and_or(uint32_t(s8 >> 32), mask, bias);
  r0[3] = and_or(uint32_t(s12), mask, bias);
  r1[3] = and_or(uint32_t(s12 >> 32), mask, bias);
  b0 = __builtin_bit_cast(bf16x8_t, r0);
  b1 = __builtin_bit_cast(bf16x8_t, r1);
}

// Position of element k%8 inside an 8-element chunk of the LDS activation
// rows: chunk order is (x0, x4, x1, x5, x2, x6, x3, x7).
__device__ __forceinline__ uint32_t chunk_pos(uint32_t k) {
  return (k & ~7u) | ((k & 3u) << 1) | ((k >> 2) & 1u);
}

// Same map applied to four packed u8 row indices at once.
__device__ __forceinline__ uint32_t chunk_pos4(uint32_t k4) {
  return and_or(k4, 0xF8F8F8F8u, and_or(k4 << 1, 0x06060606u, (k4 >> 2) & 0x01010101u));
}

// 16 bytes of X (x0..x7) -> chunk order (x0,x4,x1,x5,x2,x6,x3,x7): one byte
// permute per output dword.
__device__ __forceinline__ uint4 permute_chunk(uint4 w) {
  uint4 o;
  o.x = __builtin_amdgcn_perm(w.z, w.x, 0x05040100u);   // x0 | x4 << 16
  o.y = __builtin_amdgcn_perm(w.z, w.x, 0x07060302u);   // x1 | x5 << 16
  o.z = __builtin_amdgcn_perm(w.w, w.y, 0x05040100u);   // x2 | x6 << 16
  o.w = __builtin_amdgcn_perm(w.w, w.y, 0x07060302u);   // x3 | x7 << 16
  return o;
}

// ---------------------------------------------------------------------------
// One Tile-COO group (16 bytes, four slots), decoded as the paper's outlier
// decoding step describes (Sec. 4.2): four u8 rows, four u8 columns, four
// bf16 values; value bits 0x0000 mark a padding slot.
// ---------------------------------------------------------------------------
struct Group {
  uint32_t rows;   // k0 | k1 << 8 | k2 << 16 | k3 << 24 (tile-local)
  uint32_t cols;   // n0 | n1 << 8 | n2 << 16 | n3 << 24 (tile-local)
  uint32_t v01;    // bf16 v0 | v1 << 16
  uint32_t v23;    // bf16 v2 | v3 << 16
};

__device__ __forceinline__ Group decode_group(uint4 g) {
  Group d;
  d.rows = g.x;
  d.cols = g.y;
  d.v01 = g.z;
  d.v23 = g.w;
  return d;
}

__device__ __forceinline__ uint32_t slot_row(const Group& d, int j) { return (d.rows >> (8 * j)) & 0xFFu; }
__device__ __forceinline__ uint32_t slot_col(const Group& d, int j) { return (d.cols >> (8 * j)) & 0xFFu; }
__device__ __forceinline__ uint32_t slot_val(const Group& d, int j) {
  return ((j < 2 ? d.v01 : d.v23) >> (16 * (j & 1))) & 0xFFFFu;
}
// All four slots in one column (always true in by-column mode).
__device__ __forceinline__ bool single_column(const Group& d) {
  return d.cols == (d.cols & 0xFFu) * 0x01010101u;
}

// ---------------------------------------------------------------------------
// Number formats.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits) {
  return __builtin_bit_cast(float, bits << 16);
}

__device__ __forceinline__ float f16_bits_to_f32(uint32_t bits) {
  return float(__builtin_bit_cast(_Float16, uint16_t(bits)));
}

// fp32 -> bf16, round to nearest, ties to even (IEEE 754 rounding applied to
// the 16 dropped bits); NaN stays a quiet NaN.
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return ((u >> 16) | 0x40u) & 0xFFFFu;
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                         __builtin_bit_cast(bf16x2_t, b), c, false);
}

// ---------------------------------------------------------------------------
// Global loads, waits.
// ---------------------------------------------------------------------------
// Every operand is read with raw buffer loads: a resource descriptor per
// array (base and byte size, wave-uniform), a per-lane byte offset fixed for
// the whole kernel, and a wave-uniform byte offset that moves from tile to
// tile.  Address arithmetic therefore stays in scalar registers; the plan
// keeps every array below 2^31 bytes.
constexpr int kBufferWord3 = 0x00020000;   // raw 32-bit elements, no swizzle (gfx9)
constexpr int kSc1 = 16;                   // cache-policy operand: device (agent) scope

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, int(bytes), kBufferWord3);
}

__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, int(voff), int(soff), 0));
}
__device__ __forceinline__ uint2 buf_load8(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), 0));
}
__device__ __forceinline__ uint32_t buf_load4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), 0);
}

// Calls f(integral_constant<int, I>) for I = B .. E-1, in order.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt low bits [3:0], high bits [15:14]; expcnt and lgkmcnt left at max).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// ---------------------------------------------------------------------------
// The outlier image.
// ---------------------------------------------------------------------------
// MFMA mode: the B-operand image of a strip's tile (128 rows x 16 NCB
// columns).  Local column n' of the strip belongs to MFMA column block
// j = n' % NCB at position c = n' / NCB, so element (k, n') is read by lane
// (c + 16 * ((k%32)/8)) as B of MFMA (step k/32, block j), at the position its
// X partner holds k (chunk order x0,x4,x1,x5,...).  As a bf16 index into the
// wave's image its bits are, for 64-column strips (NCB = 4, 16 KB image)
//   0: k2 | 1-2: k0,k1 | 3-6: n'2..n'5 | 7-8: k3,k4 | 9-10: n'0,n'1 | 11-12: k5,k6
// and for 32-column strips (NCB = 2, 8 KB image)
//   0: k2 | 1-2: k0,k1 | 3-6: n'1..n'4 | 7-8: k3,k4 | 9: n'0 | 10-11: k5,k6.
// image_offsets forms the four byte offsets of a group at once, one slot per
// byte lane while the index is split into its low and high bytes, then two
// slots per dword (16-bit halves; the offsets are below 2^14).  C holds the
// Tile-COO columns (0..63); a 32-column strip uses their low five bits.
template <int NCB>
__device__ __forceinline__ void image_offsets(uint32_t R, uint32_t C, uint32_t& o01, uint32_t& o23) {
  const uint32_t r1 = R << 1, r2 = R >> 2;
  uint32_t lo = r2 & 0x01010101u;               // k2
  lo = and_or(r1, 0x06060606u, lo);             // k0, k1
  uint32_t hi = (R >> 4) & 0x01010101u;         // k4
  if constexpr (NCB == 4) {
    const uint32_t c1 = C << 1;
    lo = and_or(c1, 0x78787878u, lo);           // n'2..n'5
    hi = and_or(c1, 0x06060606u, hi);           // n'0, n'1
    hi = and_or(r2, 0x18181818u, hi);           // k5, k6
  } else {
    lo = and_or(C << 2, 0x78787878u, lo);       // n'1..n'4
    hi = and_or(C << 1, 0x02020202u, hi);       // n'0
    hi = and_or(R >> 3, 0x0C0C0C0Cu, hi);       // k5, k6
  }
  lo = and_or(R << 4, 0x80808080u, lo);         // k3
  // [lo0 hi0 lo1 hi1] and [lo2 hi2 lo3 hi3], then element -> byte offset
  o01 = __builtin_amdgcn_perm(hi, lo, 0x05010400u) << 1;
  o23 = __builtin_amdgcn_perm(hi, lo, 0x07030602u) << 1;
}

// The same slots as full LDS byte addresses, for images that lie below
// 64 KB of LDS at a 256-byte-aligned base: the byte-lane assembly builds byte
// offsets (the bit layouts above shifted up by one) and ORs the base's high
// byte, replicated in `base_rep`, into the high bytes, where its bits lie
// above the offset's.  Each 16-bit half is then a whole address.
template <int NCB>
__device__ __forceinline__ void image_addresses(uint32_t R, uint32_t C, uint32_t base_rep,
                                                uint32_t& a01, uint32_t& a23) {
  const uint32_t r1 = R >> 1, r3 = R >> 3;
  uint32_t lo = r1 & 0x02020202u;                 // k2
  lo = and_or(R << 2, 0x0C0C0C0Cu, lo);           // k0, k1
  uint32_t hi = and_or(r3, 0x03030303u, base_rep);   // k3, k4
  if constexpr (NCB == 4) {
    const uint32_t c2 = C << 2;
    lo = and_or(c2, 0xF0F0F0F0u, lo);             // n'2..n'5
    hi = and_or(c2, 0x0C0C0C0Cu, hi);             // n'0, n'1
    hi = and_or(r1, 0x30303030u, hi);             // k5, k6
  } else {
    lo = and_or(C << 3, 0xF0F0F0F0u, lo);         // n'1..n'4
    hi = and_or(C << 2, 0x04040404u, hi);         // n'0
    hi = and_or(R >> 2, 0x18181818u, hi);         // k5, k6
  }
  a01 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
  a23 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
}

typedef __attribute__((address_space(3))) uint16_t lds_u16;

// 16-bit LDS store at an absolute LDS byte address.
__device__ __forceinline__ void lds_store16(uint32_t addr, uint32_t v) {
  *reinterpret_cast<lds_u16*>(uintptr_t(addr)) = uint16_t(v);
}

// LDS byte address where a dynamic-LDS pointer points.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return uint32_t(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) const unsigned char*)(p)));
}

// Writes a group's four values into the image at absolute LDS address `img`
// and returns where they went.  A padding slot (value bits 0) goes to the
// trash word instead, since its position may coincide with a real element of
// another group, and so does a slot whose column lies in the other half of a
// 64-column Tile-COO tile when the strip is 32 columns wide (`half` = which
// half this strip is; bit 5 of a column selects the half).
// With FA the addresses come whole from image_addresses (`img` then holds
// the replicated base byte instead of the base).
template <int NCB, bool FA>
__device__ __forceinline__ void group_addresses(uint32_t img, uint32_t R, uint32_t C,
                                                uint32_t o[4]) {
  uint32_t o01, o23;
  if constexpr (FA) {
    image_addresses<NCB>(R, C, img, o01, o23);
    o[0] = o01 & 0xFFFFu;
    o[1] = o01 >> 16;
    o[2] = o23 & 0xFFFFu;
    o[3] = o23 >> 16;
  } else {
    image_offsets<NCB>(R, C, o01, o23);
    o[0] = img + (o01 & 0xFFFFu);
    o[1] = img + (o01 >> 16);
    o[2] = img + (o23 & 0xFFFFu);
    o[3] = img + (o23 >> 16);
  }
}

__device__ __forceinline__ void store_group(const uint32_t addr[4], uint4 raw) {
  lds_store16(addr[0], raw.z);
  lds_store16(addr[1], raw.z >> 16);
  lds_store16(addr[2], raw.w);
  lds_store16(addr[3], raw.w >> 16);
}

typedef uint16_t u16x2_t __attribute__((__vector_size__(2 * sizeof(uint16_t))));

// 0xFFFF in each 16-bit half of v that is not zero, else 0.  (In assembly: the
// compiler would turn it back into comparisons.)
__device__ __forceinline__ uint32_t nonzero_halves(uint32_t v) {
  uint32_t n;
  asm("v_pk_min_u16 %0, %1, 1 op_sel_hi:[1,0]" : "=v"(n) : "v"(v));
  asm("v_pk_sub_i16 %0, 0, %1" : "=v"(n) : "v"(n));
  return n;
}

// Bytes of 0 or 1 -> bytes of 0 or 0xFF (m * 255, without the multiplication).
__device__ __forceinline__ uint32_t spread_bytes(uint32_t m) {
  uint32_t r;
  asm("v_lshlrev_b32 %0, 8, %1" : "=v"(r) : "v"(m));
  return r - m;
}

// mask ? a : b, bit by bit (truth table 0xCA).
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA);
}

// Which of a group's slots are written to an image, as 0xFFFF / 0 halves
// (slots 0, 1 in m01; 2, 3 in m23): the value is not padding and, for NCB = 2,
// bit 5 of the column equals `half`.  Masks in vector registers instead of
// comparisons, whose conditions the scalar unit puts together for v_cndmask: with
// comparisons the row-block kernel takes 34.6 us (4096 x 14336 at 128 rows), here
// 33.3, and 36.1 (4096 x 28672 at 64 rows), here 35.0; 32-column strips 7.10 (4096 x
// 4096 at one row), here 6.97, and 7.59 at 8 rows, here 7.47; 64-column strips the same.
template <int NCB>
__device__ __forceinline__ void slot_masks(uint4 raw, uint32_t half, uint32_t& m01, uint32_t& m23) {
  uint32_t v01 = raw.z, v23 = raw.w;
  if constexpr (NCB == 2) {
    // one byte per slot, 1 where the half matches, spread to 0xFF
    const uint32_t m = ((raw.y >> 5) ^ ((half ^ 1u) * 0x01010101u)) & 0x01010101u;
    const uint32_t mm = spread_bytes(m);
    v01 &= __builtin_amdgcn_perm(mm, mm, 0x01010000u);
    v23 &= __builtin_amdgcn_perm(mm, mm, 0x03030202u);
  }
  m01 = nonzero_halves(v01);
  m23 = nonzero_halves(v23);
}

template <int NCB, bool FA>
__device__ __forceinline__ void scatter_group(uint32_t img, uint32_t trash, uint4 raw,
                                              uint32_t half, uint32_t use, uint32_t addr[4]) {
  uint32_t o[4], m01, m23;
  group_addresses<NCB, FA>(img, raw.x, raw.y, o);
  slot_masks<NCB>(raw, half, m01, m23);
  m01 &= use;   // all ones, or zero: every slot to the trash word
  m23 &= use;
  addr[0] = bit_select(uint32_t(int32_t(m01 << 16) >> 16), o[0], trash);
  addr[1] = bit_select(uint32_t(int32_t(m01) >> 16), o[1], trash);
  addr[2] = bit_select(uint32_t(int32_t(m23 << 16) >> 16), o[2], trash);
  addr[3] = bit_select(uint32_t(int32_t(m23) >> 16), o[3], trash);
  store_group(addr, raw);
}

__device__ __forceinline__ void clear_group(const uint32_t addr[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) lds_store16(addr[j], 0u);
}

}  // namespace fqk

// Fused outlier-aware W4A16 matmul for more than 16 rows and a long K (gfx950):
// the row-block kernel.
//
// The strip kernel (kernels.hip) gives every wave its own tiles, X slice and
// outlier image, at most 32 rows at a time: with many rows it spends its time
// on repeated work -- every 32-row slab dequantises the weights, builds the
// outlier image and stages X for 64 columns again.  Here a workgroup computes
// a block of 32 RB rows (RB = 1 or 2) x 128 columns, and its waves share X:
//
//   waves     eight, as two K groups (kKG) of four column waves (kCW).  A K
//             group walks its half of the workgroup's tiles; a column wave
//             computes all rows x 32 columns with v_mfma_f32_32x32x16_bf16.
//   turns     two waves share a SIMD, one of each K group, and the groups run
//             half a tile apart: while one multiplies a tile (32 RB / 2 MFMAs of
//             32 cycles, dequantisation and the staging of X between them), the
//             other scales the tile before into its sums and scatters the
//             outliers of the next.  Two barriers a tile keep them in step.
//             Both groups multiplying at once left the MFMAs idle while both
//             scaled: 35.9 against 34.1 us (4096 x 14336 at 128 rows).
//   X         the group's 32 RB x 128 slice of a tile is loaded row-wise, 16
//             bytes per lane, 2 RB loads per wave, one tile ahead; permuted to
//             the order of the dequantised codes and stored to one of two LDS
//             buffers while the other is read.  Its row sums, which eq. (3)
//             needs, come from one MFMA chain per wave and tile, each column
//             wave summing one 16-row block for all four.
//   codes     8 bytes per lane and 32-row step (2 adjacent columns), two tiles
//             ahead, dequantised in registers as in the strip kernel after one
//             v_permlane16_swap per step.
//   outliers  each wave scatters its 32 columns' half of the Tile-COO tile into
//             an image of its own (8 KB), right after the image of the tile
//             before has been read and cleared.
//   reduce    the two K groups add their halves through LDS, each finishing
//             half of the rows; with split-K each workgroup stores its sums in
//             register order with device-coherent stores and the last to
//             arrive at the block's counter adds them in split order.
//
// What bounds it: the issue of one wave's turn.  With 64 rows a turn takes 0.76
// to 0.83 us (the instrumented build's tile loop over its turns), about 2000
// cycles at 2.4 GHz: 1088 of MFMA (32 of 32 cycles, 4 of 16), and LDS reads, waits
// and the other instructions that do not fit between them.
// Per call, strip kernel -> this one (1 % outliers, graph replay, rotated weights,
// both in turn in one process):
//   4096 x 28672  128 rows 79.1 -> 65.1 us, 64 rows 47.6 -> 34.1, 27 rows 27.3 -> 24.8
//   4096 x 14336  128 rows 45.8 -> 33.1 us, 64 rows 26.0 -> 22.2, 40 rows 25.2 -> 21.8
//   14336 x 4096  128 rows 39.6 -> 33.6 us, 64 rows 25.7 -> 23.6
//   4096 x 6144   128 rows 24.8 -> 21.4 us
// With two group loads per tile (64 rows only; 5 % outliers): 4096 x 14336 at 128 rows
// 49.0 -> 37.2 us, at 64 rows 27.7 -> 24.7.
// Tried and slower (4096 x 14336 at 128 rows, 34.1 us then): 16x16x32 MFMAs 38.2 us
// with scalar-unit masks in the scatter; tile_indptr by scalar loads, which every
// LDS wait then waits for, 39.0 us; all loads and the scatter's addresses among
// the MFMAs 39.0 us; X stored one step later or earlier 34.8 and 36.0 us; LDS
// fragments two steps ahead 34.8 us; the row sums in the scaling turn 35.2 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace fqk {

namespace {

constexpr int kCW = 4;                       // column waves per K group
constexpr int kKG = 2;                       // K groups per workgroup
constexpr int kRowsCols = 32 * kCW;          // columns of a workgroup's block
constexpr int kRowsImage = 8192;             // outlier image of 128 x 32, bytes
constexpr int kRowsGBits = 20;               // as the strip kernel packs G and S

typedef float f32x16_t __attribute__((__vector_size__(16 * sizeof(float))));

struct RowsTail {
  int y_f32;
  const uint4* packed;
  int64_t n_groups;
  void* Y;
  float* partials;
  uint32_t* counters;
#ifdef FQ_WAVE_STAMPS
  uint64_t* stamps;
#endif
};

#ifdef FQ_WAVE_STAMPS
// A wave's start, its first tile's X and groups in LDS, its last turn's end, its exit.
__device__ __forceinline__ void store_stamps(const RowsTail& tail, int tid, uint64_t s0, uint64_t s1,
                                             uint64_t s2) {
  const uint64_t s3 = __builtin_amdgcn_s_memrealtime();
  const uint32_t w = blockIdx.x * uint32_t(kCW * kKG) + uint32_t(tid >> 6);
  if ((tid & 63) == 0 && tail.stamps && w < uint32_t(fqi::kMaxStampWaves)) {
    tail.stamps[4 * w] = s0;
    tail.stamps[4 * w + 1] = s1;
    tail.stamps[4 * w + 2] = s2;
    tail.stamps[4 * w + 3] = s3;
  }
}
#endif

// LDS layout, bytes, one 64 KB page per K group: the group's images, the
// waves' trash words, its row sums and its first X buffer (image and trash of
// a wave in one page, so that the scatter works on packed 16-bit addresses);
// the second X buffers follow the last page.  The K groups' exchange at the
// end takes the images' place.
template <int RB>
struct RowsLds {
  static constexpr int kRows = 32 * RB;
  static constexpr int kPage = 65536;
  static constexpr int kXBuf = kRows * 256;
  static constexpr int off_trash = kCW * kRowsImage;
  static constexpr int off_sum = off_trash + kCW * 16;
  static constexpr int off_x = off_sum + kRows * 4;
  static constexpr int off_x1 = (kKG - 1) * kPage + off_x + kXBuf;
  static constexpr int off_flag = off_x1 + kKG * kXBuf;
  static constexpr int bytes = off_flag + 16;
  static_assert(off_x + kXBuf <= kPage && off_x % 16 == 0, "a group's page");
  static_assert(kCW * RB * 4 * 1024 <= off_trash, "the K groups' exchange fits the images");
};

// One tile's codes, scales and zero-points of a wave's 32 columns.
struct RowsTile {
  uint2 w[4];
  uint32_t s, z;
};

// LDS writes of this wave are done, then all waves meet.  Global loads stay
// in flight (no wait on the vector-memory counter).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The B operand of v_mfma_f32_32x32x16_bf16 holds column lane % 32 and the
// 8 k-consecutive values of packed row lane / 32.  A lane loads two adjacent
// columns of one packed row (lane (c4, h): columns 2 c4, 2 c4 + 1 of row 4 s + h);
// swapping odd 16-lane rows of the first word with even ones of the second
// turns the two words into two operands: lanes 0-15 column 2 c4, lanes 16-31
// column 2 c4 + 1, of packed rows 4 s (lanes 0-31) and 4 s + 2 (first operand),
// or 4 s + 1 and 4 s + 3 (second).
//
// The outlier image is that operand: block 2 s + m (1 KB), then lane, then the
// eight values in the order of the dequantised codes.  Byte offset bits:
//   1: k2 | 2-3: k0,k1 | 4-7: n'1..n'4 | 8: n'0 | 9: k4 | 10: k3 | 11-12: k5,k6
// (n' the column within the 32, m = k3, s = k5,k6).  The four slots' addresses
// within the 64 KB page, two to a dword; base_rep holds the image's high
// address byte in every byte.
__device__ __forceinline__ void rows_addresses(uint32_t R, uint32_t C, uint32_t base_rep,
                                               uint32_t& a01, uint32_t& a23) {
  const uint32_t r1 = R >> 1, r2 = R >> 2;
  uint32_t lo = r1 & 0x02020202u;                  // k2
  lo = and_or(R << 2, 0x0C0C0C0Cu, lo);            // k0, k1
  lo = and_or(C << 3, 0xF0F0F0F0u, lo);            // n'1..n'4
  uint32_t hi = and_or(C, 0x01010101u, base_rep);  // n'0
  hi = and_or(R >> 3, 0x02020202u, hi);            // k4
  hi = and_or(r1, 0x04040404u, hi);                // k3
  hi = and_or(r2, 0x18181818u, hi);                // k5, k6
  a01 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
  a23 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
}

// Where a group's four values go: their places, or the trash word (trash_rep,
// its address within the page in both halves) for a slot that is not this
// image's; everything to the trash word with use = 0.
__device__ __forceinline__ void rows_places(uint32_t page, uint32_t base_rep, uint32_t trash_rep,
                                            uint4 raw, uint32_t half, uint32_t use,
                                            uint32_t addr[4]) {
  uint32_t a01, a23, m01, m23;
  rows_addresses(raw.x, raw.y, base_rep, a01, a23);
  slot_masks<2>(raw, half, m01, m23);
  a01 = bit_select(m01 & use, a01, trash_rep);
  a23 = bit_select(m23 & use, a23, trash_rep);
  addr[0] = __builtin_amdgcn_perm(page, a01, 0x07060100u);
  addr[1] = __builtin_amdgcn_perm(page, a01, 0x07060302u);
  addr[2] = __builtin_amdgcn_perm(page, a23, 0x07060100u);
  addr[3] = __builtin_amdgcn_perm(page, a23, 0x07060302u);
}

template <int RB, bool SPARSE, int GL>
__global__ void __launch_bounds__(64 * kCW * kKG) __attribute__((amdgpu_waves_per_eu(2)))
rows_kernel(const uint32_t* Wq, const uint16_t* scales, const uint32_t* zeros, const uint16_t* X,
            const uint32_t* tile_indptr, int M_all, int K, int N, int GS, RowsTail tail) {
  typedef RowsLds<RB> L;
  extern __shared__ __align__(16) unsigned char smem[];
#ifdef FQ_WAVE_STAMPS
  const uint64_t stamp0 = __builtin_amdgcn_s_memrealtime();
#endif
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / kCW, cw = wave % kCW;
  const int h = lane >> 4, c4 = lane & 15;
  const int l32 = lane & 31, kh = lane >> 5;

  // Work: as in the strip kernel, workgroups are dealt round-robin to the
  // XCDs, each XCD gets a contiguous run of (column block, split) pairs, and
  // the row blocks of one pair follow one another on the same XCD.
  const int G = GS & ((1 << kRowsGBits) - 1), S = GS >> kRowsGBits;
  const int T = K >> 7;
  const int n_blocks = (M_all + L::kRows - 1) / L::kRows;
  const int bid = blockIdx.x;
  int wg, rb;
  if ((G & 7) == 0) {
    const int t = bid >> 3;
    rb = t % n_blocks;
    wg = (bid & 7) * (G >> 3) + t / n_blocks;
  } else {
    rb = bid / G;
    wg = bid - rb * G;
  }
  const int cb = wg / S, sp = wg - cb * S;   // column block, split
  const int m0 = rb * L::kRows;
  const int M = min(L::kRows, M_all - m0);
  const int t_lo = int(uint32_t(sp * T) / uint32_t(S));
  const int t_hi = int(uint32_t((sp + 1) * T) / uint32_t(S));
  const int iters = (t_hi - t_lo + kKG - 1) / kKG;   // group 0's tiles, the larger half
  const int w_lo = min(t_lo + kg * iters, t_hi - 1);   // (a group without tiles reads the last one)
  const int cnt = max(0, min(iters, t_hi - t_lo - kg * iters));   // this group's tiles
  const int last = max(cnt, 1) - 1;                  // past it that tile is read again

  // A wave whose columns lie past N (N is a multiple of 64) computes the last
  // 32 columns again and stores nothing.
  const bool in_n = cb * kRowsCols + 32 * cw < N;
  const int n0 = in_n ? cb * kRowsCols + 32 * cw : N - 32;
  const uint32_t half = uint32_t(n0 >> 5) & 1u;      // which half of its Tile-COO tile

  const __amdgpu_buffer_rsrc_t rw = make_rsrc(Wq, uint32_t(K / 8) * uint32_t(N) * 4u);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales, uint32_t(T) * uint32_t(N) * 2u);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(zeros, uint32_t(T) * uint32_t(N / 8) * 4u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + size_t(m0) * K, uint32_t(M) * uint32_t(K) * 2u);
  // this lane's column in the MFMA result, scales and zero-points
  const int col = 2 * c4 + (h & 1);
  const uint32_t ls = uint32_t(col) * 2u, lz = uint32_t(col >> 3) * 4u;
  const int zsh = (col & 7) * 4;
  uint32_t lw[4];   // packed row 4 step + h, columns 2 c4, 2 c4 + 1
#pragma unroll
  for (int step = 0; step < 4; ++step) lw[step] = uint32_t((4 * step + h) * N + 2 * c4) * 4u;
  uint32_t lx[2 * RB];   // staging: row 16 j + 4 cw + h, chunk c4; rows past M read row M-1
#pragma unroll
  for (int j = 0; j < 2 * RB; ++j)
    lx[j] = (uint32_t(min(16 * j + 4 * cw + h, M - 1)) * uint32_t(K) + 8u * uint32_t(c4)) * 2u;

  unsigned char* const page_p = smem + kg * L::kPage;
  unsigned char* const img_p = page_p + cw * kRowsImage;
  const uint32_t page = lds_address(page_p);   // dynamic LDS starts at 0: a multiple of 64 KB
  const uint32_t img_rep = uint32_t(cw * (kRowsImage >> 8)) * 0x01010101u;
  const uint32_t trash_rep = uint32_t(L::off_trash + cw * 16) * 0x00010001u;
  unsigned char* const xbuf[2] = {page_p + L::off_x, smem + L::off_x1 + kg * L::kXBuf};
  float* const sums = reinterpret_cast<float*>(page_p + L::off_sum);

  // Byte offsets of the tile whose loads go out next, advanced tile by tile
  // up to the group's last.
  int next = 0;
  uint32_t ox = uint32_t(w_lo) * 256u;
  uint32_t ow = (uint32_t(w_lo) * 16u * uint32_t(N) + uint32_t(n0)) * 4u;
  uint32_t os = (uint32_t(w_lo) * uint32_t(N) + uint32_t(n0)) * 2u;
  uint32_t oz = (uint32_t(w_lo) * uint32_t(N >> 3) + uint32_t(n0 >> 3)) * 4u;
  auto advance = [&]() __attribute__((always_inline)) {
    const bool go = next < last;
    ++next;
    ox += go ? 256u : 0u;
    ow += go ? uint32_t(N) * 64u : 0u;
    os += go ? uint32_t(N) * 2u : 0u;
    oz += go ? uint32_t(N) >> 1 : 0u;
  };
  auto load_codes = [&](RowsTile& r) __attribute__((always_inline)) {
#pragma unroll
    for (int step = 0; step < 4; ++step) r.w[step] = buf_load8(rw, lw[step], ow);
    r.s = uint32_t(__builtin_amdgcn_raw_buffer_load_b16(rs, int(ls), int(os), 0));
    r.z = buf_load4(rz, lz, oz);
  };
  uint4 xr[2 * RB];
  auto load_x = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2 * RB; ++j) xr[j] = buf_load16(rx, lx[j], ox);
  };
  // The loaded slice into one of the group's buffers, 16-byte chunk q of row r
  // at q ^ (r % 16): 16 lanes touch 16 distinct bank groups both here and when
  // a fragment is read.
  const uint32_t x_store = uint32_t(4 * cw + h) * 256u + (uint32_t(c4 ^ (4 * cw + h)) << 4);
  auto store_x = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2 * RB; ++j)
      *reinterpret_cast<uint4*>(xbuf[b] + j * 4096 + x_store) = permute_chunk(xr[j]);
  };

  // The tiles' group offsets: lane i holds that of the group's tile i (at most
  // 63 tiles per K group, the plan sees to it).
  const uint32_t ng = uint32_t(tail.n_groups);
  uint32_t tp = 0;
  __amdgpu_buffer_rsrc_t rg = rw;
  if (SPARSE) {
    tp = tile_indptr[uint32_t(n0 >> 6) * uint32_t(T) + uint32_t(w_lo + min(lane, last + 1))];
    rg = make_rsrc(tail.packed, max(ng, 1u) * 16u);
  }
  uint4 gr[GL] = {};               // groups lane + 64 j of a tile
  uint32_t g_lo = 0, g_n = 0;      // range of the tile whose groups are in gr
  auto load_groups = [&](int i) __attribute__((always_inline)) {
    const int t = min(i, last);
    g_lo = min(uint32_t(__builtin_amdgcn_readlane(int(tp), t)), ng);
    const uint32_t g_hi = max(g_lo, min(uint32_t(__builtin_amdgcn_readlane(int(tp), t + 1)), ng));
    g_n = i < cnt ? g_hi - g_lo : 0u;   // past the group's last tile: no groups
#pragma unroll
    for (int j = 0; j < GL; ++j)
      gr[j] = buf_load16(rg, min(uint32_t(lane + 64 * j), g_n ? g_n - 1 : 0u) * 16u, g_lo * 16u);
  };
  // The loaded groups go into the (all-zero) image in two steps: where their
  // values go, which needs no LDS and is begun among a tile's MFMAs (36.7 us in
  // one step against 34.2), and the stores.  Lanes past the last group rewrite
  // it; an empty tile's loaded group is not its own and goes to the trash
  // word.  The only branch is the one to the rare tile of more than
  // 64 GL groups, whose others are loaded here.
  uint32_t addr[GL][4] = {}, next_addr[GL][4];
  uint32_t s_n = 0;                // groups that the image holds
  auto place = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < GL; ++j)
      rows_places(page, img_rep, trash_rep, gr[j], half, g_n ? 0xFFFFFFFFu : 0u, next_addr[j]);
  };
  auto scatter = [&]() __attribute__((always_inline)) {
    s_n = g_n;
#pragma unroll
    for (int j = 0; j < GL; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) addr[j][e] = next_addr[j][e];
      store_group(addr[j], gr[j]);
    }
    if (__builtin_expect(s_n > 64u * GL, 0)) {
      for (uint32_t g0 = 64 * GL; g0 < s_n; g0 += 64) {   // the last group again past the end
        const uint4 raw = buf_load16(rg, min(g0 + lane, s_n - 1) * 16u, g_lo * 16u);
        uint32_t ad[4];
        rows_places(page, img_rep, trash_rep, raw, half, 0xFFFFFFFFu, ad);
        store_group(ad, raw);
      }
    }
  };
  // Zeros again: at the places written, or everywhere where more than one
  // pass of groups was.
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < GL; ++j) clear_group(addr[j]);
    if (__builtin_expect(s_n > 64u * GL, 0)) {
      uint4* b4 = reinterpret_cast<uint4*>(img_p);
#pragma unroll
      for (int i = 0; i < kRowsImage / 1024; ++i) b4[i * 64 + lane] = uint4{0u, 0u, 0u, 0u};
    }
  };

  f32x16_t acc[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[b][q] = 0.f;

  // Fragments of 32-row step s: A[m][b] of packed rows 4 s + m + 2 kh and row
  // block b, and the image's blocks.
  bf16x8_t A[2][2][RB], Bo[2][2];
  const uint32_t a_row = uint32_t(l32) * 256u;
  uint32_t a_off[4][2];   // within a 32-row block, per (s, m)
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int m = 0; m < 2; ++m) a_off[s][m] = a_row + (uint32_t((4 * s + m + 2 * kh) ^ c4) << 4);
  auto fetch = [&](int buf, int s, int p) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
      for (int b = 0; b < RB; ++b)
        A[p][m][b] = *reinterpret_cast<const bf16x8_t*>(xbuf[buf] + b * 8192 + a_off[s][m]);
      if (SPARSE)
        Bo[p][m] = __builtin_bit_cast(
            bf16x8_t, reinterpret_cast<const uint4*>(img_p)[(2 * s + m) * 64 + lane]);
    }
  };

  // Every tile's loads go out in the order X, groups, codes, here and in the
  // loop, so that each wait leaves the following tile's in flight.
  RowsTile rt[2];
  load_x();
  __builtin_amdgcn_sched_barrier(0);
  if (SPARSE) load_groups(0);
  load_codes(rt[0]);
  advance();
  __builtin_amdgcn_sched_barrier(0);
  if (SPARSE) {
    uint4* b4 = reinterpret_cast<uint4*>(img_p);
#pragma unroll
    for (int i = 0; i < kRowsImage / 1024; ++i) b4[i * 64 + lane] = uint4{0u, 0u, 0u, 0u};
  }
  store_x(0);
  load_x();
  __builtin_amdgcn_sched_barrier(0);
  if (SPARSE) {
    place();
    scatter();
    load_groups(1);
  }
  load_codes(rt[1]);
  advance();
  __builtin_amdgcn_sched_barrier(0);

  const bf16x8_t ones = __builtin_bit_cast(
      bf16x8_t, u32x4_t{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
  const int sb = min(cw, 2 * RB - 1);      // the 16-row block whose sums this wave makes
  auto body = [&](int i, auto bc) __attribute__((always_inline)) {
    constexpr int B = decltype(bc)::value;   // code registers and X buffer of tile i
    RowsTile& r = rt[B];
    f32x16_t tmp[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) tmp[b][q] = 0.f;
    bf16x8_t As[4];
    f32x4_t xsum{0.f, 0.f, 0.f, 0.f};
    // The other group's turn to scale ends here.  No wait comes with it: of this
    // wave's LDS reads only those of a tile's first X and image blocks may be out,
    // which nothing overwrites before the next lds_barrier.  The row sums, which
    // the next tile overwrites, have been read: their use in the scaling is not
    // moved past the barrier.
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int p = s & 1;
      if (s < 3) fetch(B, s + 1, p ^ 1);
      As[s] = *reinterpret_cast<const bf16x8_t*>(xbuf[B] + sb * 4096 + c4 * 256 +
                                                 (((4 * s + h) ^ c4) << 4));
      // columns 2 c4 and 2 c4 + 1 of one packed row -> the two operands
      const auto sw = __builtin_amdgcn_permlane16_swap(r.w[s].x, r.w[s].y, false, false);
      bf16x8_t Bq[2];
      dequant_pair<true>(sw[0], sw[1], Bq[0], Bq[1]);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        if (SPARSE) {
#pragma unroll
          for (int b = 0; b < RB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[p][m][b], Bo[p][m], acc[b], 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < RB; ++b)
          tmp[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[p][m][b], Bq[m], tmp[b], 0, 0, 0);
      }
      if (SPARSE && s == 1) place();
      if (s == 2) {
        store_x(B ^ 1);
        load_x();
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
      xsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(As[s], ones, xsum, 0, 0, 0);
    // every column of the result is the sum: 16 lanes store the same value
    *reinterpret_cast<f32x4_t*>(sums + 16 * sb + 4 * h) = xsum;
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    f32x4_t xs[4 * RB];
#pragma unroll
    for (int q = 0; q < 4 * RB; ++q)
      xs[q] = *reinterpret_cast<const f32x4_t*>(sums + 8 * q + 4 * kh);
    if (SPARSE) {
      clear();
      scatter();
      load_groups(i + 2);
    }
    // eq. (3) once per (group, column), in fp32.  A group that is one tile
    // short multiplies its last tile again with scale zero (and no outliers).
    const float sc = f16_bits_to_f32(i < cnt ? r.s : 0u);
    const float nz = -(kCodeOffset + float((r.z >> zsh) & 15u));
#pragma unroll
    for (int q = 0; q < 4 * RB; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[q / 4][4 * (q % 4) + e] += sc * (tmp[q / 4][4 * (q % 4) + e] + nz * xs[q][e]);
    load_codes(r);
    advance();
    fetch(B ^ 1, 0, 0);   // the next tile's first step
  };
  // The K groups run half a tile apart: while one multiplies, the other, on
  // the same SIMDs, stages, scatters and scales.
  lds_barrier();   // the first X slices
#ifdef FQ_WAVE_STAMPS
  const uint64_t stamp1 = __builtin_amdgcn_s_memrealtime();
#endif
  fetch(0, 0, 0);
  if (kg == 1) asm volatile("s_barrier" ::: "memory");
  // (pairs of tiles, then an odd last one: no path leads from an even tile to
  // the next even one, so the compiler's load counts stay exact)
  int i = 0;
  for (; i + 2 <= iters; i += 2) {
    body(i, std::integral_constant<int, 0>{});
    body(i + 1, std::integral_constant<int, 1>{});
  }
  if (i < iters) body(i, std::integral_constant<int, 0>{});
  if (kg == 0) asm volatile("s_barrier" ::: "memory");
#ifdef FQ_WAVE_STAMPS
  const uint64_t stamp2 = __builtin_amdgcn_s_memrealtime();
#endif

  // ------------------------------------------------------------------ reduce
  const int y_f32 = tail.y_f32;
  const int n_cb = (N + kRowsCols - 1) / kRowsCols;
  const uint32_t block = uint32_t(rb * n_cb + cb);
  constexpr uint32_t kPart = kCW * RB * 4 * 1024u;   // one workgroup's sums, bytes
  const __amdgpu_buffer_rsrc_t prs =
      make_rsrc(tail.partials, uint32_t(n_blocks) * uint32_t(n_cb) * uint32_t(S) * kPart);
  int* flag = reinterpret_cast<int*>(smem + L::off_flag);
  f32x4_t* ex = reinterpret_cast<f32x4_t*>(smem) + cw * RB * 4 * 64 + lane;

  // Quad qd of the accumulators: rows 8 qd + 4 kh .. + 3 of column `col`.
  // Two rows of two lanes' columns are exchanged so that each lane stores two
  // adjacent columns of one row.
  auto store_quad = [&](int qd, const f32x4_t& v) __attribute__((always_inline)) {
    if (!in_n) return;
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      const float v0 = v[e], v1 = v[e + 1];
      const auto sw = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v0),
                                                       __builtin_bit_cast(uint32_t, v1), false, false);
      const uint32_t u0 = sw[0], u1 = sw[1];
      const float a = __builtin_bit_cast(float, u0), b = __builtin_bit_cast(float, u1);
      const int row = 8 * qd + 4 * kh + e + (h & 1);
      if (row >= M) continue;
      const size_t idx = size_t(m0 + row) * N + n0 + 2 * c4;
      if (y_f32)
        *reinterpret_cast<float2*>(static_cast<float*>(tail.Y) + idx) = float2{a, b};
      else
        *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(tail.Y) + idx) =
            f32_to_bf16_rne(a) | (f32_to_bf16_rne(b) << 16);
    }
  };

  // Group 0 finishes the first half of the quads, group 1 the second.
  constexpr int kHalf = 2 * RB;
  f32x4_t mine[kHalf];
  __syncthreads();   // every wave is done with the images
#pragma unroll
  for (int q = 0; q < 4 * RB; ++q) {
    const f32x4_t v = {acc[q / 4][4 * (q % 4)], acc[q / 4][4 * (q % 4) + 1],
                       acc[q / 4][4 * (q % 4) + 2], acc[q / 4][4 * (q % 4) + 3]};
    if ((q < kHalf) == (kg == 0)) mine[q % kHalf] = v;
    else ex[q * 64] = v;
  }
  __syncthreads();
  const int q0 = kg * kHalf;
#pragma unroll
  for (int q = 0; q < kHalf; ++q) {
    mine[q] += ex[(q0 + q) * 64];   // two terms: the order does not matter
    if (S == 1) {
      store_quad(q0 + q, mine[q]);
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(u32x4_t, mine[q]), prs,
          int((block * uint32_t(S) + uint32_t(sp)) * kPart + uint32_t(cw * RB * 4 + q0 + q) * 1024u +
              uint32_t(lane) * 16u), 0, kSc1);
    }
  }
  if (S == 1) {
#ifdef FQ_WAVE_STAMPS
    store_stamps(tail, tid, stamp0, stamp1, stamp2);
#endif
    return;
  }
  __builtin_amdgcn_s_waitcnt(0);   // this thread's partial stores have completed
  __syncthreads();
  if (tid == 0) {
    const uint32_t old = __hip_atomic_fetch_add(tail.counters + block, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
    *flag = (old == uint32_t(S - 1));
  }
  __syncthreads();
  if (*flag) {
    // The last to arrive adds the partials in split order.
    const uint32_t base = block * uint32_t(S) * kPart + uint32_t(cw * RB * 4 + q0) * 1024u + uint32_t(lane) * 16u;
#pragma unroll
    for (int q = 0; q < kHalf; ++q) mine[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int kBatch = 2;
    for (int s0 = 0; s0 < S; s0 += kBatch) {
      u32x4_t part[kBatch][kHalf];
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int q = 0; q < kHalf; ++q)   // in range; surplus loads unused
          part[j][q] = __builtin_amdgcn_raw_buffer_load_b128(
              prs, int(base + uint32_t(min(s0 + j, S - 1)) * kPart + uint32_t(q) * 1024u), 0, kSc1);
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (s0 + j < S) {
#pragma unroll
          for (int q = 0; q < kHalf; ++q) mine[q] += __builtin_bit_cast(f32x4_t, part[j][q]);
        }
    }
#pragma unroll
    for (int q = 0; q < kHalf; ++q) store_quad(q0 + q, mine[q]);
    if (tid == 0)
      __hip_atomic_store(tail.counters + block, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#ifdef FQ_WAVE_STAMPS
  store_stamps(tail, tid, stamp0, stamp1, stamp2);
#endif
}

template <int RB, bool SPARSE, int GL>
int launch_rows_variant(const fqi::Plan& pl, const fqi::MatmulPtrs& p, hipStream_t stream) {
  auto kern = rows_kernel<RB, SPARSE, GL>;
  constexpr int lds = RowsLds<RB>::bytes;
  static_assert(lds <= 160 * 1024, "LDS of one CU");
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return int(e);
  RowsTail tail;
  tail.y_f32 = p.y_f32;
  tail.packed = reinterpret_cast<const uint4*>(p.packed);
  tail.n_groups = p.n_groups;
  tail.Y = p.Y;
  tail.counters = static_cast<uint32_t*>(p.workspace);
  tail.partials = reinterpret_cast<float*>(static_cast<char*>(p.workspace) + fqi::kCounterRegion);
#ifdef FQ_WAVE_STAMPS
  tail.stamps = fqi::wave_stamps_address();
#endif
  const int G = pl.rows_G, S = pl.rows_S;
  hipLaunchKernelGGL(kern, dim3(unsigned(G) * unsigned(pl.rows_blocks)), dim3(64 * kCW * kKG), lds,
                     stream, p.Wq, p.scales, p.zeros, p.X, p.tile_indptr, pl.M, pl.K, pl.N,
                     G | (S << kRowsGBits), tail);
  return int(hipGetLastError());
}

}  // namespace

}  // namespace fqk

namespace fqi {

// Whether the row-block kernel is faster than the strip kernel's plan `p`, for rb
// 32-row blocks per workgroup, S K ranges, units blocks of Y and so many rounds of
// workgroups.  Figures: strip kernel's time over the row-block kernel's (above 1 the
// latter is faster), graph replay, rotated weights, at K x N and the rows given.
//
// Measure: `strips` workgroups of the strip kernel on the busiest CU (two run at a
// time), each with tiles of up to 32 rows x 64 columns, against this kernel's rounds;
// x = theirs / ours, the strip tiles of a CU per tile of this kernel, of which four
// cover a tile of 64 rows x 128 columns.
//
// 64-row blocks with outliers (a tile takes 0.775 us, a strip tile 0.29): from x = 3
// on, with a split, whose partial sums cost about 3 us, from 3.5.  At x = 2 -- 65 to
// 96 rows and 8192 < N <= 10880, half of the CUs and at most 3/4 of the rows used --
// 4096 x 8576 0.82 to 0.84, 14336 x 8576 0.74 to 0.76, 4096 x 10880 0.85; at x = 3
// 4096 x 11008 at 65 rows 1.10, split 17280 x 4352 0.95.  More than eight K ranges
// also need x = 5 or two strip workgroups on a CU (28672 x 2048, 16 ranges, x = 4: 0.92
// to 0.96; 28672 x 1024 at 65 to 96 rows, two per CU, 1.14 to 1.19).
//
// 64-row blocks without outliers (0.635 against 0.19 us): from x = 3.5 on (4096 x
// 28672 at 112 rows 1.04, at 33 1.16); from 3.3 up to 20 tiles (2560 x 38400 1.05;
// 4096 x 38400 0.97); from 3 in a single round up to 24 tiles, 18 where the last block
// has at most 16 rows (2688 x 22336 at 33 rows 1.07, 4096 x 16512 0.93; 2560 x 11008 at
// 65 rows 0.96).  With a split from x = 5 on; at x = 4 where the strip kernel splits
// too on two workgroups per CU (14336 x 2048 at 65 to 96 rows 1.14 to 1.20), with a
// nearly full last block from 20 tiles on (5120 x 13824 at 64 rows 1.11), and from 28
// where two strip workgroups share a CU (8192 x 11008 at 33 rows 1.05; 4096 x 11008, 16
// tiles, 0.95; 14336 x 4096 at 65 rows, one per CU, 0.91).
//
// 32-row blocks do the work of the two strip workgroups that they replace and save
// one start: 25 to 32 rows up to 80 tiles (8192 x 28672 at 28 rows 1.04, 12288 x 16512
// 0.99); up to 24 rows, where strip tiles stage less X, up to 40 tiles, 24 where fewer
// than 140 CUs get a block (4096 x 18432 to 24576 1.02 to 1.05, 4096 x 16512 0.98 to
// 1.00, 8192 x 16512 0.96).  Without outliers up to 64 tiles from 21 rows on (8192 x
// 20480 at 24 rows 1.10), below up to 24 (4096 x 28672 at 17 rows 0.93).
static bool rows_faster(const Plan& p, int rb, int blocks, int S, int64_t units, int64_t rounds,
                        bool outliers) {
  if (rb == 1)
    return p.T <= (p.M > 24 ? 80 : units < 140 ? 24 : outliers ? 40 : p.M > 20 ? 64 : 24);
  const int64_t strips = (int64_t(p.G) * p.n_slabs + 255) / 256;
  const int64_t theirs = strips * S, ours = rounds * p.S;
  if (outliers) {
    if (S == 1) return theirs >= 3 * ours;
    return 2 * theirs >= 7 * ours && (S <= 8 || theirs >= 5 * ours || strips >= 2);
  }
  const int tiles = p.T / S, last = p.M - 64 * (blocks - 1);   // rows of the last block
  if (S == 1)
    return 2 * theirs >= 7 * ours || (3 * theirs >= 10 * ours && tiles <= 20) ||
           (rounds == 1 && theirs >= 3 * ours && tiles <= (last > 16 ? 24 : 18));
  if (theirs >= 5 * ours) return true;
  if (theirs < 4 * ours) return false;
  return (strips >= 2 && (p.S > 1 || tiles >= 28)) || (last > 48 && tiles >= 20);
}

// The row-block kernel's launch for a problem the strip kernel's plan accepts:
// blocks of 64 rows, 32 up to 32 rows.  The split fills the CUs with one
// workgroup each.
// It takes the calls that rows_faster gives it, where every workgroup has at
// least kRowsMinTiles tiles: below, its start (two tiles of loads, an LDS exchange)
// and the partial sums of the larger blocks cost more than the shared work
// saves (64 rows: 14336 x 4096, 14 tiles, 23.6 against 25.7 us; 4096 x 6144, 6
// tiles, 17.4 against 16.7; 4096 x 4096, 4 tiles, 16.9 against 13.9.  128 rows:
// 4096 x 4096, 8 tiles, 17.8 against 16.8; 4096 x 6144, 16 tiles, 21.4 against
// 24.8).  Up to 32 rows only without a split (27 rows: 4096 x 28672 24.8 against
// 27.3 us, 4096 x 14336 split 2 18.6 against 18.5).
// A matrix with a tile of more than kRowsMaxGroups groups is left to the strip
// kernel, whose waves do not wait for one another at every tile (5 % outliers,
// half in 2 % of the columns, over 200 groups in a tile: 4096 x 14336 at 128 rows
// 70.7 against 62.7 us; 2 %, 100 to 150 groups, at 64 rows: 26.7 against 32.1).  With
// 32-row blocks, whose turns are too short to cover a second load or the wait of a
// fuller tile, already one of more than kRowsMaxGroups32 (3 %, up to 79 groups: 3328 x
// 25792 at 17 rows 27.0 against 23.4, 4096 x 28672 at 32 rows 32.4 against 30.1; 5 %:
// 26.9 against 23.8, 32.8 against 31.5; 2 %, half in 2 % of the columns, up to 139: 30.6
// against 23.5, 33.5 against 30.5.  2 % uniform, up to 55: 21.9 against 22.5, 26.9
// against 30.4).
// More than one round of workgroups has to be filled, in CUs and rows together, by
// kRowsMinFill (4096 x 38400 at 64 rows, 300 workgroups, 0.59: 68.9 against 62.6 us;
// 4096 x 28672 at 80 rows, 0.55: 67.6 against 67.7, at 128 rows, 0.88: 65.1 against
// 79.1); up to 32 rows only a single round gains (8192 x 57344 at 32 rows 98.4
// against 97.2).
// Partial sums beyond kRowsPartialLimit are left to the strip kernel, so that
// every default launch fits the static scratch.
void plan_rows(Plan* p, bool outliers) {
  p->rows_RB = 0;
  if (p->M <= kRowsMinM) return;
  const int rb = p->M <= 32 ? 1 : 2;
  if (p->max_tile_groups > (rb == 1 ? kRowsMaxGroups32 : kRowsMaxGroups)) return;
  const int blocks = (p->M + 32 * rb - 1) / (32 * rb);
  const int n_cb = (p->N + fqk::kRowsCols - 1) / fqk::kRowsCols;
  const int64_t units = int64_t(n_cb) * blocks;
  int S = int(std::max<int64_t>(1, 256 / units));
  if (rb == 1 && S > 1) return;
  S = std::max(S, (p->T + 125) / 126);   // at most 63 tiles per K group
  if (p->T / S < kRowsMinTiles) return;
  // one workgroup runs per CU: rounds of 256
  const int64_t wgs = units * S, rounds = (wgs + 255) / 256;
  if (rounds > 1 && rb == 1) return;
  if (rounds > 1 && double(wgs) / double(256 * rounds) * p->M / (32 * rb * blocks) < kRowsMinFill) return;
  if (!rows_faster(*p, rb, blocks, S, units, rounds, outliers)) return;
  const int64_t part = S > 1 ? units * S * fqk::kCW * rb * 4 * 1024 : 0;
  if (part > int64_t(kRowsPartialLimit)) return;
  if (int64_t(n_cb) * S >= (1 << fqk::kRowsGBits) || units > kMaxStrips) return;
  p->rows_RB = rb;
  p->rows_blocks = blocks;
  p->rows_S = S;
  p->rows_G = n_cb * S;
  p->rows_partial_bytes = size_t(part);
  p->ws_bytes = std::max(p->ws_bytes, kCounterRegion + size_t(part));
}

size_t rows_lds_bytes(const Plan& pl) {
  return pl.rows_RB == 1 ? size_t(fqk::RowsLds<1>::bytes) : size_t(fqk::RowsLds<2>::bytes);
}

int launch_rows(const Plan& pl, const MatmulPtrs& p, bool sparse, bool two_group_loads, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (pl.rows_RB == 1) {
    if (!sparse) return fqk::launch_rows_variant<1, false, 1>(pl, p, s);
    return fqk::launch_rows_variant<1, true, 1>(pl, p, s);   // tiles of one load, plan_rows sees to it
  }
  if (!sparse) return fqk::launch_rows_variant<2, false, 1>(pl, p, s);
  return two_group_loads ? fqk::launch_rows_variant<2, true, 2>(pl, p, s)
                         : fqk::launch_rows_variant<2, true, 1>(pl, p, s);
}

}  // namespace fqi

// Table-tile kernels: the LDS-resident, wide-gather formulation of the lookup-MAC loop.
//
// The layer is acc[i][j] = sum_k LUT(A[i][k], B[k][j])  (Sec. II Eq. (3) with the product
// taken from the truth table; Sec. III "matrix multiplication phase").  One operand is put
// on the lanes (index i, one or more elements per lane), the other on small per-step
// tables (index j):
//
//   for a tap k and a group of 8 columns j..j+7, the workgroup builds in LDS a table of 256
//   entries of 16 bytes, entry v = the eight 16-bit products LUT(v, B[k][j..j+7]);
//   every lane element's entry A[i][k] is fetched with ONE 16-byte LDS read, and a matrix instruction
//   adds the bytes of 128 such entries (16 elements, eight taps) to int32 accumulators.
//
// So a lookup-MAC costs 2 bytes of LDS read bandwidth and a 1024th of a matrix instruction, instead of
// one conflict-prone 2-byte gather and an addition per MAC.  The 128 kB truth table itself stays in L2:
// the tables are assembled from a row-major re-layout of it ("rows": for each code of the
// table-side operand the 256 products against every lane-side code, 512 contiguous bytes),
// read with coalesced global loads that do not compete with the LDS gathers.
//
// Two lane assignments share the kernel:
//   variant 2  lanes = output pixels   (A = im2col view of x, B = filters, rows = LUT^T)
//   variant 3  lanes = output channels (A = filters^T, B = im2col(x)^T, rows = LUT)
// Work is divided over the grid by (tile, chunk) iterations rather than by tiles, so that all
// compute units stay busy whatever the layer shape; tiles shared by several workgroups are
// combined by a small fix-up kernel (integer addition is associative: same bits).
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

#include "ax_internal.h"

namespace ax {

constexpr int kChunk = 16;     // taps per 16-byte lane-operand load

// Quantization values in the form the table-tile kernels consume, in device memory: prep_kernel
// derives them from the call's host parameters or from device-resident coefficients.
struct QDev {
  int32_t z_lane, z_tab;  // zero points of the lane-side and of the table-side operand
  long long kzz;          // K * z_lane * z_tab
  float scale;            // x_scale * w_scale
  uint32_t pad4;          // pad code in all four bytes
  uint32_t pad_[2];
  uint32_t padrow[4];     // sixteen pad codes (16-byte aligned): what a tap outside the image reads
};
static_assert(sizeof(QDev) == 48 && offsetof(QDev, padrow) == 32, "padrow must be 16-byte aligned");

// i / d = umulhi(2 i, mul) >> shift for 0 <= i < 2^31: mul = ceil(2^(31 + shift) / d) with shift = ceil(log2 d) is at most
// 2^32 - 1, and too large by less than d / (2^(31 + shift)) of the quotient's unit, which 2 i < 2^32 leaves under one.
// (A division by a variable is some thirty dependent instructions, in 64 bits a hundred and more.)
struct Divisor {
  uint32_t mul;
  int shift;
  Divisor() = default;
  explicit Divisor(int d) : mul(0), shift(0) {
    while ((1LL << shift) < d) ++shift;
    mul = (uint32_t)(((1ull << (31 + shift)) + d - 1) / d);
  }
  __device__ __forceinline__ int operator()(int i) const { return (int)(__umulhi(2u * (uint32_t)i, mul) >> shift); }
};

struct TabArgs {
  // lane-side operand, addressed as an implicit im2col view of an [N,H,W,Cin] tensor
  const uint8_t* A;
  int I;   // valid lane elements
  int ih;  // lane elements per tile (multiple of 64, at most the kernel's tile height)
  int H, W, Cin, KW, sh, sw, ph, pw, OHW, OW;
  Divisor by_ohw, by_ow, by_cin, by_kw, by_ntiles1, by_ntj;
  // byte offset of the 16 codes (pixel, channels ci0 .. ci0+15) = pixel * a_ps + ci0 * a_cs:
  // (Cin, 1) for a tensor read in place; (16, I) for materialized patches, which lie chunk by
  // chunk ([K16 / 16][I][16]) so that the lanes of a wave read one contiguous kilobyte
  uint32_t a_ps, a_cs;
  // table-side operand, packed [Krows][Jpad] with zero fill
  const uint8_t* Bp;
  int Jpad, J;
  const int32_t* bsum;   // [nseg][Jpad] partial column sums of Bp (k segments), see prep_kernel
  int nseg;
  const uint16_t* rows;  // re-laid-out truth table, 256 rows of 512 bytes
  int K;
  // work decomposition: tile t = ti * ntj + tj, nch chunks of 16 taps per tile; workgroup w of G
  // takes iterations [w*total/G, (w+1)*total/G) of the tile-major iteration space
  int ntj, nch;
  long long total_iters;
  int small;                    // total_iters below 2^31 and G at most 46340: shares and tiles by 32-bit arithmetic:
  int share, rest;              // total_iters = share * G + rest
  Divisor by_grid, by_nch;
  const struct QDev* qd;  // zero points, scale and pad code as the kernels use them (written by prep_kernel)
  int dh, dw;        // dilation of the implicit im2col view
  uint32_t bias_k;   // 32768 * K for signed tables (their entries are stored with that offset), else 0
  int32_t* acc_out;
  float* y_out;
  int32_t* part;  // [2*G][ih * kJT] partial tiles: slot 2w = workgroup w's piece of a tile begun by
                  // another workgroup, slot 2w+1 = its piece of a tile it begins but does not end
  int32_t* lsum;  // [2*G][ih] lane-operand sums of the same pieces
  uint32_t* cnt;  // non-null: [tiles] arrival counters, pieces are combined inside tab_kernel (see there)
  const uint4* tabs;  // kernels with PRE: [nch][Jpad/8][256][16] ready-made table entries (prep_tables_kernel)
  uint32_t tabs_bytes;
  long long out_elems;   // outputs per table (M * Cout)
  int ntiles1;           // tiles of one table; tile index space = table * ntiles1 + tile (several tables: ax_conv2d_multi_lut)
  int vec_out;  // outputs may be written along j in aligned pieces of 8 bytes (1), of 16 bytes (2)
  int padded;   // 0: every tap of every pixel lies in the image, 1: not, 2: not and positions need more than 16 bits
  int xcd;      // 1: shares of work are numbered XCD by XCD (see xcd_major), 0: in launch order
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 512;           // 8 waves of up to 256 registers
constexpr int kWaves = kThreads / 64;
constexpr int kGroups = 8;              // most groups of 64 lane elements per wave
constexpr int kIT = kThreads * kGroups; // lane elements of a full tile
constexpr int kJT = 8;                  // columns of a tile: one 16-byte table entry
constexpr int kTabBytes = 65536;        // tables of one chunk: 256 entries x 16 taps x 16 bytes

// Position of workgroup b of a grid of G when the workgroups are listed XCD by XCD (workgroup b
// runs on XCD b % 8): a bijection of 0 .. G-1.
__device__ __forceinline__ int xcd_major(int b, int G) {
  const int x = b & 7, q = G >> 3, r = G & 7;
  return x * q + min(x, r) + (b >> 3);
}

// A 64-bit value that is the same in all lanes, in scalar registers (its arithmetic may be done in vector ones).
__device__ __forceinline__ long long uniform(long long v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((unsigned long long)v >> 32));
  return (long long)((unsigned long long)hi << 32 | lo);
}

// Column constants K z_lane z_tab - z_lane * (column sum) of a tile's eight columns, into red[THREADS / 64][8]
// (the sum over its rows is a column's constant): thread = (segment, column), so that the loads of
// all segments (kMaxSeg at most) are in flight together.  The caller has a barrier before the constants are read.
constexpr int kMaxSeg = 64;  // segments of the table-side column sums
template <int THREADS>
__device__ __forceinline__ int32_t column_sum_part(const TabArgs& a, int j0, int tid) {
  int32_t sb = 0;
#pragma unroll
  for (int s = 0; s < kMaxSeg; s += THREADS / 8) {
    const int seg = s + (tid >> 3);
    if (seg < a.nseg) sb += a.bsum[(size_t)seg * a.Jpad + j0 + (tid & 7)];
  }
  return sb;
}
template <int THREADS>
__device__ __forceinline__ void column_constants(int32_t sb, long long kzz, int z_lane, int tid, long long (*red)[8]) {
#pragma unroll
  for (int o = 8; o < 64; o *= 2) sb += __shfl_xor(sb, o);
  if ((tid & 63) < 8) red[tid >> 6][tid & 7] = (tid < 8 ? kzz : 0LL) - (long long)z_lane * sb;
}
template <int WAVES>
__device__ __forceinline__ long long column_constant(const long long (*red)[8], int col) {
  long long t = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) t += red[w][col];
  return t;
}

// What a piece or a finished tile holds per (group of 64 lane elements, quarter r of it): lane
// l = 16 kg + m has columns 2 kg and 2 kg + 1 of lane element 16 r + m.
__device__ __forceinline__ float dequant(uint32_t accv, uint32_t lterm, long long cterm, float scale, bool wide) {
  // accv - lterm + cterm is the corrected sum; every term is below 2^31 in magnitude, and so is
  // every partial sum for K <= 16384: 32-bit wrap-around arithmetic is exact.  Longer K takes 64 bits.
  return wide ? (float)((long long)(int32_t)(accv - lterm) + cterm) * scale
              : (float)(int32_t)(accv - lterm + (uint32_t)cterm) * scale;
}

// Outputs of one lane: columns j, j + 1 (j = tile column 2 kg) of lane element i.
template <bool CH>
__device__ __forceinline__ void put_pair(const TabArgs& a, int32_t* acc_base, float* y_base, int i, int j, uint32_t v0,
                                         uint32_t v1, float y0, float y1) {
  if (!CH && a.vec_out) {
    if (j < a.J) {
      const size_t o = (size_t)i * a.J + j;
      if (acc_base) *reinterpret_cast<uint2*>(acc_base + o) = make_uint2(v0, v1);
      if (y_base) *reinterpret_cast<float2*>(y_base + o) = make_float2(y0, y1);
    }
  } else {
    const size_t o = CH ? (size_t)j * a.I + i : (size_t)i * a.J + j;
    const size_t step = CH ? (size_t)a.I : (size_t)1;
    if (j < a.J) {
      if (acc_base) acc_base[o] = (int32_t)v0;
      if (y_base) y_base[o] = y0;
    }
    if (j + 1 < a.J) {
      if (acc_base) acc_base[o + step] = (int32_t)v1;
      if (y_base) y_base[o + step] = y1;
    }
  }
}

// One workgroup of 8 waves per compute unit; a tile is up to 4096 lane elements x 8 columns.
// CH: lanes are output channels (output index j*I + i) instead of pixels (i*J + j).
//
// Gathers and sums.  The wave's 64 lanes are 16 lane elements (m = lane % 16) times four taps
// (kg = lane / 16): every lane fetches the entry of ITS element's code at ITS tap, 16 bytes = eight
// products; two such fetches are what v_smfmac_i32_16x16x128_i8 takes from a lane as 32 contraction elements
// of column m.  The other operand is a constant: row r of it picks byte r of every 16, so the instruction adds,
// for 16 lane elements at once, the low and the high bytes of the eight products over eight
// taps: one matrix instruction per 1024 lookups where adding in vector registers takes
// sixteen vector instructions.  A row has one value in every 16, so the sparse form (two of every four) holds it and
// takes twice the bytes of v_mfma_i32_16x16x64_i8 in the same 16 clocks: with that one a phase of a full tile was 4096
// clocks of matrix instructions per SIMD beside 4096 of gathers, and the two do not overlap fully: a full tile took a
// tenth longer, 512 elements a fiftieth.  The bytes count as signed, so the tables hold every
// byte with its top bit flipped (value - 128) and the epilogue adds 128 * (1 + 256) per tap.
//
// Table layout.  LDS holds two buffers of 16 tables, interleaved entry by entry: entry v of tap t
// lies at 256 v + 16 t, so the bank of a gather depends on the tap alone.  The LDS serves a 16-byte
// read in passes of 16 lanes that are not consecutive: measured times single out lanes 0-3, 12-15,
// 20-23 and 24-27 of 32 (and their complement), two quarters from each of two neighbouring kg.  A
// pass is therefore free of conflicts, whatever the codes are, when its 16 lanes are at 16
// different taps: lane (kg, m) walks the four taps of dword dq of its element's sixteen codes in the order
// s ^ (m % 4), with dq = kg where m / 4 is even and kg ^ 2 where it is odd.  (With the tables one after another
// and random codes in the bank index, gathers took 1.6-2.2 times as long; with dq = kg ^ (m / 4)
// 1.5 times.  Full rotations kg ^ 0, 2, 3, 1 are free of conflicts too, but take eight selects per group of 64
// elements to turn the codes, these four: a hundredth of a phase of a full tile, three ready-made.)
// The address is one byte permute: byte 1 is the code, byte 0 the constant 16 t.
//
// Work is spread over the grid by iterations, not by tiles (G workgroups, one per compute
// unit, each takes an equal contiguous share of tiles x chunks): a workgroup runs through one or
// more "segments" (a tile and a chunk range of it).  A segment that covers its tile's whole K
// range writes final outputs; any other writes a partial tile that tab_fixup_kernel combines.
// Integer addition is associative, so the decomposition does not change a single bit.
//
// A phase is one chunk of 16 taps: the waves gather from one buffer and fill the other with the
// tables of the next chunk, then meet at a barrier.  Without PRE a wave builds 32 entries of all 16
// tables: lane = (tap, quarter), eight 16-byte loads (one per column, from the 512-byte row of the
// column's code; the four lanes of a tap read 64 contiguous bytes), interleaved and stored entry by entry.
// Of the two waves of a SIMD one stores its entries and requests the next rows before it gathers, the other (late)
// requests its rows first and stores after its gathers: one keeps the vector unit and the LDS writes busy while the
// other one's gathers keep the LDS reads and the matrix unit, and their row requests do not queue up behind each other.
// With the dense matrix instruction, the entries of all waves stored between their gathers and the rows requested before
// the barrier a phase took 1.24 us at 512 elements, 1.53 at 1024, 1.83 at 1600, 2.36 at 2112, 2.90 at 3136 and 3.51 at
// 4096; so it takes 0.98, 1.24, 1.58, 1.94, 2.55 and 3.11, ready-made 1.39, 1.56, 1.68, 2.15, 2.52 and 2.86 (the copies come
// from beyond the L2s; side by side on one device).  The rows of 64 KB of tables alone take 0.56 us.
// PRE: the tables of a chunk lie ready-made in global memory as an image of the LDS buffer
// (prep_tables_kernel) and are copied straight into LDS (buffer loads with the lds modifier).
//
// What a segment costs beside its phases: shares, tiles and pixels are found by multiplication (Divisor), the column
// constants and coefficients are requested with the first tables instead of after the last phase, and nothing is
// requested past the last chunk where the tables are ready-made: 100352 x 16 x 256 (1024 tiles of one phase, one
// output) 75 -> 61 us, 100352 x 64 x 256 115 -> 98.
//
// Bound: LDS.  Per phase of a full tile (7000 clocks) 1 MiB of gathers, 4097 clocks on their own (256 bytes per clock), and 64
// KiB of table writes, 745 (88 bytes per clock), against 2048 clocks of matrix instructions per SIMD.
// PADDED: taps may lie outside the image and read the pad row instead (operands that could not be
// copied with their border, see prep_chunks_kernel); the other form has no position per lane
// element and no comparisons.  PADDED spills 112 bytes per lane at full height, the others at most 20
// (28 x 28 x 128, 3 x 3, batch 16: 203 us in place, 91 from the copy).  All forms keep 84 to 137 scalars in lanes of vector
// registers; few of their moves lie in the loops, most where a segment begins and ends.
// GR: groups of 64 lane elements per wave.  Tiles of at most half the height take GR = 4, whose free
// registers hold the lane operands and the table rows a whole phase ahead: with few groups to gather
// a phase is shorter than a round trip to memory.
template <int GR, bool CH, bool PRE, bool PADDED>
__global__ __launch_bounds__(kThreads, 2) void tab_kernel(const TabArgs a) {
  __shared__ struct {
    alignas(16) uint8_t tab[2 * kTabBytes];  // at LDS address 0: only there the gathers' constant offsets fit
    long long cterm[kWaves][kJT];  // column constants of the current tile, see the epilogue
    int comb[3];                 // last piece of a shared tile? / first and last share of the tile
  } sh;
  constexpr int XR = PRE ? GR : GR < kGroups ? 4 : 2;  // groups whose lane operands are in registers or in flight
  constexpr int DB = !PRE && GR < kGroups ? 2 : 1;  // chunks whose table rows are
  // PADDED spills in its loop at full height, less with one role: 47 layers read in place take 0.98 of the time
  // with one, four of them 0.90 to 0.92 (12760 x 5328 x 32, 3 x 3, whose border has no room: 141.2 us, 128.5).
  constexpr bool kOneRole = PADDED && GR == kGroups;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kg = lane >> 4;
  const uint8_t* padrow = reinterpret_cast<const uint8_t*>(a.qd->padrow);
  const uint32_t lds0 = (uint32_t)(uintptr_t)sh.tab;

  // constant operand of the matrix instruction: row m has a 1 at byte m of every 16.  It is sparse, two
  // values of every four with their places in pick_at: (m % 4, 3) or, for m % 4 = 3, (0, 3).
  i32x4 pick;
  const int high = (m & 3) == 3;
#pragma unroll
  for (int d = 0; d < 4; ++d) pick[d] = (m >> 3) == (d & 1) ? 1 << (16 * (m >> 2 & 1) + 8 * high) : 0;
  const int pick_at = (high ? 0xc : 0xc | (m & 3)) * 0x11111111;
  // gather addresses: perm[s] takes byte s of offs (16 * tap) and the code of that tap
  const bool swap = m >> 2 & 1;
  uint32_t offs = 0, perm[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t b = (uint32_t)(s ^ (m & 3));
    offs |= 16u * (4u * (uint32_t)(swap ? kg ^ 2 : kg) + b) << (8 * s);
    perm[s] = 0x0c0c0000u | (4u + b) << 8 | (uint32_t)s;
  }

  // Workgroups go to the eight XCDs (each with its own L2) in turn.  With a.xcd the share of work
  // is taken by a renumbered index under which every XCD holds a contiguous run of shares:
  // neighbouring tiles read the same lane-side rows, which then come from one L2 instead of being
  // fetched into eight.  (Where tiles are cut into a multiple of eight shares the launch order
  // already gives every XCD one slice of K of all tiles; the planner picks per layer.)
  const int wg = a.xcd ? xcd_major((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x;
  auto share_begin = [&](int w) -> long long {  // w * total / G
    return a.small ? (long long)(w * a.share + __builtin_amdgcn_readfirstlane(a.by_grid(w * a.rest)))
                   : uniform((long long)w * a.total_iters / gridDim.x);
  };
  long long it_beg = share_begin(wg);
  const long long it_end = share_begin(wg + 1);

  // builder roles: tap bt, entries bv .. bv + 7
  const int bt = lane >> 2, bv = 32 * wave + 8 * (lane & 3);
  u32x4 tabs_words;  // PRE: buffer descriptor of the table images (raw buffer, bounds-checked against their size)
  tabs_words.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)a.tabs);
  tabs_words.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)((uintptr_t)a.tabs >> 32) & 0xffffu));
  tabs_words.z = (uint32_t)__builtin_amdgcn_readfirstlane((int)(PRE ? a.tabs_bytes : 0u));
  tabs_words.w = 0x00020000u;

  while (it_beg < it_end) {
  // The lane as the parts of a segment outside its main loop use it: what depends on it is computed anew for every
  // segment, where kept across the loop it would be spilled.
  int ls = lane;
  asm volatile("" : "+v"(ls));
  const int gtile = __builtin_amdgcn_readfirstlane(a.small ? a.by_nch((int)it_beg) : (int)(it_beg / a.nch));
  const int c_beg = (int)(it_beg - (long long)gtile * a.nch);
  const int tbl = __builtin_amdgcn_readfirstlane(a.by_ntiles1(gtile));  // which multiplier table
  const int tile = gtile - tbl * a.ntiles1;
  const uint16_t* __restrict__ rows = a.rows + (size_t)tbl * 65536;
  int32_t* __restrict__ acc_base = a.acc_out ? a.acc_out + (size_t)tbl * a.out_elems : nullptr;
  float* __restrict__ y_base = a.y_out ? a.y_out + (size_t)tbl * a.out_elems : nullptr;
  const int c_end = (int)min((long long)a.nch, c_beg + (it_end - it_beg));
  const bool whole = (c_beg == 0) && (c_end == a.nch);
  const int ti = __builtin_amdgcn_readfirstlane(a.by_ntj(tile));
  const int i0 = ti * a.ih;  // tiles are a.ih <= kIT lane elements high (a multiple of 64)
  const int tj = tile - ti * a.ntj;
  const int j0 = tj * kJT;

  // ---- lane operand --------------------------------------------------------------------
  // Group p of this wave is lane elements i0 + 64 * (8 p + wave) .. + 63 of the tile; groups at or
  // beyond a.ih (or beyond the operand) are padding: the first np groups are real.  For the loads
  // lane l holds element l of the group.
  const int left = min(a.ih, a.I - i0);
  const int np = max(0, ((left + 63) / 64 - wave + kWaves - 1) / kWaves);
  // Byte offset of the element from the tile's first one: pixels under tap (0, 0) come in rising order,
  // and their distance fits 32 bits (launch_tab), so a load is a scalar base and this offset.
  // PADDED: index of the pixel instead, which may lie outside the image, and its row and column, 16 bits each.
  uint32_t pix[GR];
  int yx[GR];
  auto first_tap = [&](int p, int& by, int& bx) {  // position of tap (0, 0); returns the image
    const int i = min(i0 + 64 * (kWaves * p + wave) + ls, a.I - 1);
    const int n = a.by_ohw(i);
    const int r = i - n * a.OHW;
    const int oy = a.by_ow(r);
    by = oy * a.sh - a.ph;
    bx = (r - oy * a.OW) * a.sw - a.pw;
    return n;
  };
  if (!PADDED && a.OHW == 1 && a.H == 1 && a.W == 1) {  // an element is a pixel: the copy by output pixel, the patches, the filters
#pragma unroll
    for (int p = 0; p < GR; ++p) pix[p] = (uint32_t)min(i0 + 64 * (kWaves * p + wave) + ls, a.I - 1);
  } else {
#pragma unroll
    for (int p = 0; p < GR; ++p) {
      int by, bx;
      const int n = first_tap(p, by, bx);
      pix[p] = (uint32_t)((n * a.H + by) * a.W + bx);
      if (PADDED) yx[p] = (int)((uint32_t)by * 65536u + (uint32_t)bx);
    }
  }
  uint32_t pix0 = 0;  // the pixel of the tile's first element
  if (!PADDED) {
    const int n = a.by_ohw(i0), r = i0 - n * a.OHW;
    const int oy = a.by_ow(r);
    pix0 = (uint32_t)__builtin_amdgcn_readfirstlane((n * a.H + oy * a.sh) * a.W + (r - oy * a.OW) * a.sw);
#pragma unroll
    for (int p = 0; p < GR; ++p) pix[p] = (pix[p] - pix0) * a.a_ps;
  }
  int xdy = 0, xdx = 0, xoff = 0;  // tap of the chunk that load_x reads: row and column step, pixels from tap (0, 0)
  const uint8_t* xsrc = a.A;       // its channels
  auto load_from = [&](int chunk) {
    const int k0 = min(chunk, a.nch - 1) * kChunk;
    const int tap = __builtin_amdgcn_readfirstlane(a.by_cin(k0));
    const int ky = __builtin_amdgcn_readfirstlane(a.by_kw(tap));
    xdy = ky * a.dh;
    xdx = (tap - ky * a.KW) * a.dw;
    xoff = xdy * a.W + xdx;
    xsrc = a.A + (size_t)(uint32_t)(k0 - tap * a.Cin) * a.a_cs;
    if (!PADDED) xsrc += (size_t)(pix0 + (uint32_t)xoff) * a.a_ps;
  };
  auto load_x = [&](int p) {
    // Every lane loads, also in groups of tile padding (the last element again) and, PADDED, at taps
    // outside the image (sixteen pad codes kept in device memory).  A load that only some waves
    // issued would leave the number of loads in flight unknown at compile time, and every later wait
    // for table rows would then have to wait for all loads, the activation prefetch included.
    if (!PADDED) {
      uint32_t off = pix[p];
      asm volatile("" : "+v"(off));  // stays one 32-bit register next to a scalar base
      return *reinterpret_cast<const u32x4*>(xsrc + off);
    }
    const uint8_t* src = xsrc + (size_t)(pix[p] + (uint32_t)xoff) * a.a_ps;
    {
      int by = (yx[p] >> 16) + (int)((uint32_t)yx[p] >> 15 & 1u), bx = (int)(int16_t)yx[p];
      if (a.padded == 2) first_tap(p, by, bx);  // positions beyond 16 bits
      if ((unsigned)(by + xdy) >= (unsigned)a.H || (unsigned)(bx + xdx) >= (unsigned)a.W) src = padrow;
    }
    return *reinterpret_cast<const u32x4*>(src);
  };

  // ---- table building ------------------------------------------------------------------
  const __amdgpu_buffer_rsrc_t rows_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(rows), 0, 131072, 0x00020000);
  const int c_last = a.nch - 1;
  auto load_codes = [&](int chunk) {  // the eight column codes of this lane's tap
    return *reinterpret_cast<const uint2*>(a.Bp + (size_t)(min(chunk, c_last) * kChunk + bt) * a.Jpad + j0);
  };
  u32x4 dd[DB][8];  // entries bv .. bv + 7 of the eight columns' rows; chunk c in dd[(c - c_beg) % DB]
  auto build_issue = [&](const uint2 codes, u32x4 (&d)[8]) {
    if (PRE) return;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t b = ((c < 4 ? codes.x : codes.y) >> (8 * (c & 3))) & 0xffu;
      d[c] = __builtin_amdgcn_raw_buffer_load_b128(rows_rsrc, (int)(b * 512u) + bv * 2, 0, 0);
    }
  };
  auto build_commit = [&](int e, int buf, const u32x4 (&d)[8]) {  // entry bv + e
    if (PRE) return;
    const uint32_t s = (e & 1) ? 0x07060302u : 0x05040100u;
    u32x4 v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = __builtin_amdgcn_perm(d[2 * c + 1][e >> 1], d[2 * c][e >> 1], s);
    // the four lanes of a tap write to the same four banks: odd lanes store their halves in the other
    // order (2-way instead of 4-way conflicts: about half the clocks for a phase's tables)
    const bool odd = lane & 1;
    uint8_t* const dst = &sh.tab[buf * kTabBytes + (bv + e) * 256 + bt * 16];
    *reinterpret_cast<uint2*>(dst + (odd ? 8 : 0)) = make_uint2(odd ? v[2] : v[0], odd ? v[3] : v[1]);
    *reinterpret_cast<uint2*>(dst + (odd ? 0 : 8)) = make_uint2(odd ? v[0] : v[2], odd ? v[1] : v[3]);
  };
  // PRE: half of this wave's eighth of a chunk's image into buffer buf.  The hardware writes to LDS
  // at M0 + instruction offset + 16 * lane (the instruction offset counts for the memory address and
  // for the LDS address alike).  Written as instructions: the compiler would make every later LDS
  // read wait for a copy it knows of, since it cannot tell the two table buffers apart; the waves
  // wait for their copies once, before the barrier of the phase.
  auto table_copy = [&](int chunk, int buf, int half) {
    if (!PRE) return;
    const uint32_t part = (uint32_t)(wave * (kTabBytes / kWaves) + half * (kTabBytes / kWaves / 2));
    const uint32_t soff = ((uint32_t)min(chunk, c_last) * (uint32_t)(a.Jpad >> 3) + (uint32_t)tj) * (uint32_t)kTabBytes + part;
    const uint32_t dst = lds0 + (uint32_t)(buf * kTabBytes) + part;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:3072 lds"
                 :: "s"(__builtin_amdgcn_readfirstlane((int)dst)), "v"(lane * 16), "s"(tabs_words),
                 "s"(__builtin_amdgcn_readfirstlane((int)soff)) : "memory");
  };
  auto copies_done = [&]() {
    if (PRE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };

  // ---- main loop -----------------------------------------------------------------------
  i32x4 acc[GR][4];  // [group][quarter]: bytes 4 kg .. 4 kg + 3 of the entries' sums for element 16 r + m
  uint32_t sl[GR];   // code sums of the lane's own element (element l of the group)
#pragma unroll
  for (int p = 0; p < GR; ++p) {
    sl[p] = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[p][r] = i32x4{0, 0, 0, 0};
  }
  const int n = c_end - c_beg;
  // first chunk's tables (one global round trip), then the requests the first phase relies on
  const int32_t sb = column_sum_part<kThreads>(a, j0, 64 * wave + ls);
  int none = 0;  // in a vector register: values that the compiler knows to be uniform it would wait for at once
  asm volatile("" : "+v"(none));
  const QDev* qd = a.qd + none;
  const long long kzz = qd->kzz;
  const int z_lane = qd->z_lane;
  const int z_tab_v = qd->z_tab, row0_v = rows[none], scale_v = __float_as_int(qd->scale);
  __builtin_amdgcn_sched_barrier(0);
  table_copy(c_beg, 0, 0);
  table_copy(c_beg, 0, 1);
  build_issue(load_codes(c_beg), dd[0]);
  u32x4 xn[XR];
  load_from(c_beg);
#pragma unroll
  for (int p = 0; p < XR; ++p) xn[p] = load_x(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) build_commit(e, 0, dd[0]);
  // what the epilogue needs has travelled with them
  column_constants<kThreads>(sb, kzz, z_lane, 64 * wave + ls, sh.cterm);
  const uint32_t z_tab = (uint32_t)__builtin_amdgcn_readfirstlane(z_tab_v);
  const float scale = __int_as_float(__builtin_amdgcn_readfirstlane(scale_v));
  const uint32_t klast = (uint32_t)a.nch * kChunk;
  const uint32_t padfix =
      (klast - (uint32_t)a.K) * ((uint32_t)__builtin_amdgcn_readfirstlane(row0_v) ^ 0x8080u) + a.bias_k - 32896u * klast;
  uint2 codes = load_codes(c_beg + 1), codes2 = codes;
  if (DB == 2) codes2 = load_codes(c_beg + 2);
  copies_done();
  __syncthreads();

  // One phase: gathers of chunk ch from buffer BUF, tables of the next chunk (more: there is one) into
  // the other.
  auto phase = [&](auto LATE, auto BUF, int ch, bool more) __attribute__((always_inline)) {
    constexpr bool late = decltype(LATE)::value;
    constexpr int buf = decltype(BUF)::value;
    auto entries = [&]() __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
#pragma unroll
        for (int e = 0; e < 8; ++e) build_commit(e, buf ^ 1, dd[(buf + 1) % DB]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // Rows of a later chunk, into the registers whose entries are stored.  The column codes are requested ahead of the
    // rows: loads return in order, and waiting for the codes must not mean waiting for the rows.  Past the last chunk
    // the codes are those of the last chunk again (the number of loads in flight stays known) and the rows are never used.
    auto rows_ahead = [&](int set) __attribute__((always_inline)) {
      const uint2 codes_now = codes;
      codes = load_codes(ch + (late ? 1 : 2) + DB);
      __builtin_amdgcn_sched_barrier(0);
      build_issue(codes_now, dd[set % DB]);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (late) rows_ahead(buf);
    {
#pragma unroll
      for (int p = 0; p < GR; ++p) {
        __builtin_amdgcn_sched_barrier(0);
        // Waves that are behind go first: the priority of a wave falls as it works through the phase,
        // so that the waves of a SIMD reach the barrier together instead of one after the other.
        if (p == 0) __builtin_amdgcn_s_setprio(3);
        if (p == (3 * GR + 7) / 8) __builtin_amdgcn_s_setprio(2);
        if (p == (5 * GR + 7) / 8) __builtin_amdgcn_s_setprio(1);
        if (p == (7 * GR + 7) / 8) __builtin_amdgcn_s_setprio(0);
        // (PRE waits for all its loads at the end of the phase and issues none past the last chunk.)
        if (p == 0 && more) table_copy(ch + 1, buf ^ 1, 0);
        if (p == GR / 2 && more) table_copy(ch + 1, buf ^ 1, 1);
        const u32x4 x = xn[p % XR];
        if (p + XR == GR) load_from(ch + 1);
        if (!PRE || more) xn[p % XR] = load_x((p + XR) % GR);
        __builtin_amdgcn_sched_barrier(0);
        if (!late && p == 0) {
          entries();
          rows_ahead(buf + 1);
        }
        if (p < np) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sl[p] = __builtin_amdgcn_sad_u8(x[e], 0u, sl[p]);
          // Sixteen codes per lane (element l) -> dword dq of element 16 r + m in register r of lane
          // (kg, m): trade the dwords of lanes whose dq is kg ^ 2, then transpose rows of 16 lanes against
          // registers.
          uint32_t t[4];
          {
            const uint32_t q0 = swap ? x.z : x.x, q2 = swap ? x.x : x.z, q1 = swap ? x.w : x.y, q3 = swap ? x.y : x.w;
            const auto u = __builtin_amdgcn_permlane32_swap(q0, q2, false, false);
            const auto v = __builtin_amdgcn_permlane32_swap(q1, q3, false, false);
            const auto w = __builtin_amdgcn_permlane16_swap(u[0], v[0], false, false);
            const auto z = __builtin_amdgcn_permlane16_swap(u[1], v[1], false, false);
            t[0] = w[0]; t[1] = w[1]; t[2] = z[0]; t[3] = z[1];
          }
          // Two gathers, eight taps, go into one sparse matrix instruction; two pairs are in flight or being summed.
          // The second buffer's address does not fit the instruction's 16-bit offset: its last unit
          // is in offs.
          union { i32x8 pair; i32x4 half[2]; } ring[2];
          auto issue = [&](int i) {  // pair i: step 2 (i / 4) and the one after it, of quarter i % 4
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              uint32_t addr = __builtin_amdgcn_perm(t[i & 3], buf ? offs + 0x01010101u : offs, perm[2 * (i >> 2) + h]);
              asm volatile("" : "+v"(addr));
              ring[i & 1].half[h] =
                  *(const __attribute__((address_space(3))) i32x4*)(uintptr_t)(addr + lds0 + (buf ? kTabBytes - 1u : 0u));
            }
          };
          issue(0);
          issue(1);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            acc[p][i & 3] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(pick, ring[i & 1].pair, acc[p][i & 3], pick_at, 0, 0);
            if (i + 2 < 8) issue(i + 2);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (late) entries();
      copies_done();
      __syncthreads();
    }
  };
  // Phases in pairs, an odd last one by itself: a loop with a way out between its two phases would
  // leave the compiler unsure which loads are the youngest, and it would wait for all of them.
  auto phases = [&](auto LATE) __attribute__((always_inline)) {
    constexpr bool late = decltype(LATE)::value;
    const uint2 codes1 = codes;
    codes = !late ? load_codes(c_beg + 1 + DB) : codes2;
    __builtin_amdgcn_sched_barrier(0);
    if (!late || DB == 2) build_issue(codes1, dd[1 % DB]);
    __builtin_amdgcn_sched_barrier(0);
    if (!late && DB == 2) build_issue(codes2, dd[0]);
    __builtin_amdgcn_sched_barrier(0);
    for (int ch = c_beg; ch + 1 < c_end; ch += 2) {
      phase(LATE, std::integral_constant<int, 0>(), ch, true);
      phase(LATE, std::integral_constant<int, 1>(), ch + 1, ch + 2 < c_end);
    }
    if (n & 1) phase(LATE, std::integral_constant<int, 0>(), c_end - 1, false);
  };
  // Both halves of the workgroup pass n barriers each, one at the end of every phase; the branch is uniform in a wave, and a
  // barrier counts waves wherever they reach it.  None may be added to one role alone.
  if (!PRE && (kOneRole || wave >= kWaves / 2))
    phases(std::true_type());
  else
    phases(std::false_type());

  // ---- epilogue ------------------------------------------------------------------------
  // corr = acc - z_tab*Sl - z_lane*Sb[j] + K*z_lane*z_tab.
  // Taps K .. of the last chunk exist only in materialized operands, where both codes are 0: each
  // adds the table entry (0,0) to every sum, which is taken off again; and every tap has
  // 128 + 256 * 128 too little (see above).
  uint32_t sum[GR][4][2];
#pragma unroll
  for (int p = 0; p < GR; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sum[p][r][0] = (uint32_t)acc[p][r].x + ((uint32_t)acc[p][r].y << 8);
      sum[p][r][1] = (uint32_t)acc[p][r].z + ((uint32_t)acc[p][r].w << 8);
      // here, not where it is used: carried on as its four bytes' sums it would take twice the registers
      asm volatile("" : "+v"(sum[p][r][0]), "+v"(sum[p][r][1]));
    }
  // Corrects, converts and writes the sums of group p: lane l = 16 kg + m holds columns 2 kg, 2 kg + 1 of element 16 r + m
  // in v[r], and the code sum of element l.
  const int em = ls & 15, ekg = ls >> 4;
  const bool wide = a.K > 16384;
  auto put_group = [&](int p, uint32_t (&v)[4][2], uint32_t codes_sum) __attribute__((always_inline)) {
    const long long ct0 = column_constant<kWaves>(sh.cterm, 2 * ekg), ct1 = column_constant<kWaves>(sh.cterm, 2 * ekg + 1);
    float yv[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t lterm = z_tab * (uint32_t)__shfl((int)codes_sum, 16 * r + em);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        v[r][c] -= padfix;
        yv[r][c] = dequant(v[r][c], lterm, c ? ct1 : ct0, scale, wide);
      }
    }
    if (!CH && a.vec_out == 2) {
      // Rows of 16 lanes trade quarters for columns and store 16 bytes per lane, two lanes the 32 bytes that a tile has of
      // an output row: with 8 bytes per lane the stores took as long as three phases (100352 x 64 x 256, both outputs: 118
      // us, 102 so; one output 98 and 90).
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const int i = i0 + 64 * (kWaves * p + wave) + 16 * (r + (ekg & 1)) + em, j = j0 + 4 * (ekg >> 1);
        const size_t o = (size_t)i * a.J + j;
        const bool in = i < a.I && j < a.J;
        if (acc_base) {
          const auto c0 = __builtin_amdgcn_permlane16_swap(v[r][0], v[r + 1][0], false, false);
          const auto c1 = __builtin_amdgcn_permlane16_swap(v[r][1], v[r + 1][1], false, false);
          if (in) *reinterpret_cast<uint4*>(acc_base + o) = make_uint4(c0[0], c1[0], c0[1], c1[1]);
        }
        if (y_base) {
          const auto c0 = __builtin_amdgcn_permlane16_swap(__float_as_uint(yv[r][0]), __float_as_uint(yv[r + 1][0]), false, false);
          const auto c1 = __builtin_amdgcn_permlane16_swap(__float_as_uint(yv[r][1]), __float_as_uint(yv[r + 1][1]), false, false);
          if (in) *reinterpret_cast<uint4*>(y_base + o) = make_uint4(c0[0], c1[0], c0[1], c1[1]);
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + 64 * (kWaves * p + wave) + 16 * r + em;
        if (i < a.I) put_pair<CH>(a, acc_base, y_base, i, j0 + 2 * ekg, v[r][0], v[r][1], yv[r][0], yv[r][1]);
      }
    }
  };
  if (whole) {
#pragma unroll
    for (int p = 0; p < GR; ++p)
      if (p < np) put_group(p, sum[p], sl[p]);
  } else {
    // Piece of a tile that several workgroups share, as the registers hold it: per group of 64 lane
    // elements eight runs of 64 words ([quarter][column of the pair][lane]).
    // A slot holds a.ih lane elements (the tile height) of kJT columns.
    const int slot = 2 * wg + (c_beg > 0 ? 0 : 1);
    int32_t* part = a.part + (size_t)slot * ((size_t)a.ih * kJT);
    int32_t* lsum = a.lsum + (size_t)slot * a.ih;
#pragma unroll
    for (int p = 0; p < GR; ++p) {
      if (p >= np) continue;
      const int g = kWaves * p + wave;
      int32_t* pp = part + (size_t)g * 512 + ls;
      if (a.cnt) {  // read by another workgroup of this launch: stores that go through to memory
        __hip_atomic_store(lsum + g * 64 + ls, (int32_t)sl[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int q = 0; q < 8; ++q)
          __hip_atomic_store(pp + q * 64, (int32_t)sum[p][q >> 1][q & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        lsum[g * 64 + ls] = (int32_t)sl[p];
#pragma unroll
        for (int q = 0; q < 8; ++q) pp[q * 64] = (int32_t)sum[p][q >> 1][q & 1];
      }
    }
    if (a.cnt) {
      // Combination inside this kernel: every workgroup that has stored a piece counts itself in
      // at the tile's counter, and the one that arrives last adds all pieces up and writes the outputs
      // like the owner of a whole tile.  Nobody waits for anybody.  The counter wraps to 0 with the
      // last arrival, ready for the next launch.
      // Pieces travel between workgroups on different XCDs, each with an L2 of its own, so they
      // are stored and loaded with device-scope atomic accesses, which pass through the L2s to
      // memory; a device-scope fence would instead write back and invalidate whole L2s (measured:
      // 60 % more kernel time).  A piece store is complete once the wave's store counter has run
      // out, which is awaited before the barrier that precedes the count.
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (tid == 0) {
        const long long G = gridDim.x, t_beg = (long long)gtile * a.nch;
        auto owner = [&](long long it) {  // the share w with w*total/G <= it < (w+1)*total/G
          long long w = it * G / a.total_iters;
          while ((w + 1) * a.total_iters / G <= it) ++w;
          while (w * a.total_iters / G > it) --w;
          return (int)w;
        };
        const int w_first = owner(t_beg), w_last = owner(t_beg + a.nch - 1);
        const unsigned old = atomicInc(a.cnt + gtile, (unsigned)(w_last - w_first));
        sh.comb[0] = (old == (unsigned)(w_last - w_first)) ? 1 : 0;
        sh.comb[1] = w_first;
        sh.comb[2] = w_last;
      }
      __syncthreads();
      if (sh.comb[0]) {
        // From memory, its own piece too: with the own sums kept in registers the compiler spills around the whole segment
        // (172 bytes per lane), also where no tile is cut (a tile of one chunk at full height 19.1 -> 16.2 us).  Two groups and
        // two pieces at a time, a last single group four pieces, and none read that is not added: with four groups at a
        // time and the missing ones read again, waves of six groups read eight.  Bound by these reads and, in short launches, by
        // the code around them, which more or larger steps lengthen (sums and outputs stand in it once per group of a step).
        // 356 random layers combined here 0.985 of the time (four groups; with 4 + 2 + 1: 0.997), the cut layers of
        // ResNet-50 0.99, launches of less than 18 us 0.986.
        const int w_first = sh.comb[1], w_last = sh.comb[2];
        auto add_pieces = [&](auto GROUPS, int p0) __attribute__((always_inline)) {
          constexpr int PG = decltype(GROUPS)::value;
          uint32_t v[PG][4][2], vs[PG];
#pragma unroll
          for (int p = 0; p < PG; ++p) {
            vs[p] = 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) v[p][q >> 1][q & 1] = 0;
          }
          auto add = [&](auto PIECES, int w) __attribute__((always_inline)) {  // pieces w .. of the groups from p0
            constexpr int PW = decltype(PIECES)::value;
            uint32_t t[PW][PG][9];
#pragma unroll
            for (int k = 0; k < PW; ++k) {
              const int slot_k = 2 * (w + k) + (w + k == w_first ? 1 : 0);
              const int32_t* po = a.part + (size_t)slot_k * ((size_t)a.ih * kJT) + ls;
              const int32_t* lo = a.lsum + (size_t)slot_k * a.ih + ls;
#pragma unroll
              for (int p = 0; p < PG; ++p) {
                const int g = kWaves * (p0 + p) + wave;
                t[k][p][8] = (uint32_t)__hip_atomic_load(lo + g * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int q = 0; q < 8; ++q)
                  t[k][p][q] = (uint32_t)__hip_atomic_load(po + (size_t)g * 512 + q * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
            }
#pragma unroll
            for (int k = 0; k < PW; ++k)
#pragma unroll
              for (int p = 0; p < PG; ++p) {
                vs[p] += t[k][p][8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[p][q >> 1][q & 1] += t[k][p][q];
              }
          };
          const std::integral_constant<int, 1> one{};
          const std::integral_constant<int, 2> two{};
          const std::integral_constant<int, 3> three{};
          int w = w_first;
          if constexpr (PG == 1) {
            for (; w + 3 <= w_last; w += 4) add(std::integral_constant<int, 4>(), w);
            if (w + 2 == w_last) add(three, w);
            else if (w + 1 == w_last) add(two, w);
            else if (w == w_last) add(one, w);
          } else {
            for (; w < w_last; w += 2) add(two, w);
            if (w == w_last) add(one, w);
          }
#pragma unroll
          for (int p = 0; p < PG; ++p) put_group(p0 + p, v[p], vs[p]);
        };
        int p0 = 0;
        for (; p0 + 2 <= np; p0 += 2) add_pieces(std::integral_constant<int, 2>(), p0);
        if (p0 < np) add_pieces(std::integral_constant<int, 1>(), p0);
      }
    }
  }
  it_beg += n;
  __syncthreads();  // cterm is free again
  }  // segment loop
}

// Combine the pieces of every tile that more than one workgroup worked on.  The pieces lie in the
// slots of consecutive workgroups, as the registers of tab_kernel held them (see TabArgs::part).  A
// block takes one group of 64 lane elements of a tile, a thread one quarter of it: its lane's pair
// of columns.
// Bound: memory round trips, a block reads a few kilobytes.  So the loads of four pieces are issued
// before the first is waited for, those of the constants after them, and which workgroups share the
// tile is found with 32-bit divisions where the numbers allow it (SMALL): 25.7 MB of pieces
// (3136 x 8, four per tile) 22 -> 17 us.
template <bool CH, bool SMALL>
__global__ __launch_bounds__(256) void tab_fixup_kernel(const TabArgs a, int G, int ntiles) {
  const int groups = a.ih / 64;
  const int block = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int gtile = block / groups;
  const int g = block - gtile * groups;
  if (gtile >= ntiles) return;  // uniform; the last row of the launch is filled up
  auto owner = [&](auto it) {  // the workgroup w with w*total/G <= it < (w+1)*total/G
    const decltype(it) total = (decltype(it))a.total_iters;
    auto w = it * G / total;
    while ((w + 1) * total / G <= it) ++w;
    while (w * total / G > it) --w;
    return (int)w;
  };
  int w_first, w_last;
  if (SMALL) {
    w_first = owner((uint32_t)gtile * (uint32_t)a.nch);
    w_last = owner((uint32_t)gtile * (uint32_t)a.nch + (uint32_t)a.nch - 1u);
  } else {
    w_first = owner((long long)gtile * a.nch);
    w_last = owner((long long)gtile * a.nch + a.nch - 1);
  }
  if (w_first == w_last) return;  // finished inside tab_kernel
  const int tbl = gtile / a.ntiles1;
  const int tile = gtile - tbl * a.ntiles1;
  const uint16_t* __restrict__ rows = a.rows + (size_t)tbl * 65536;
  int32_t* __restrict__ acc_base = a.acc_out ? a.acc_out + (size_t)tbl * a.out_elems : nullptr;
  float* __restrict__ y_base = a.y_out ? a.y_out + (size_t)tbl * a.out_elems : nullptr;
  const int ti = tile / a.ntj;
  const int i0 = ti * a.ih, j0 = (tile - ti * a.ntj) * kJT;
  if (i0 + 64 * g >= a.I) return;
  __shared__ long long cterm[4][kJT];
  const int t = threadIdx.x, lane = t & 63, r = t >> 6;
  const int m = lane & 15, kg = lane >> 4;
  uint32_t v0 = 0, v1 = 0, sl = 0;
  const size_t piece = (size_t)a.ih * kJT;
  const int32_t* part = a.part + (size_t)g * 512 + r * 128 + lane;
  const int32_t* lsum = a.lsum + g * 64 + 16 * r + m;
  for (int w = w_first; w <= w_last; w += 4) {
    uint32_t p0[4], p1[4], ps[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // past the last piece: the last one again, not added
      const int wk = min(w + k, w_last);
      const int slot = 2 * wk + (wk == w_first ? 1 : 0);
      const int32_t* pp = part + (size_t)slot * piece;
      p0[k] = (uint32_t)pp[0];
      p1[k] = (uint32_t)pp[64];
      ps[k] = (uint32_t)lsum[(size_t)slot * a.ih];
    }
    if (w == w_first) column_constants<256>(column_sum_part<256>(a, j0, t), a.qd->kzz, a.qd->z_lane, t, cterm);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t on = w + k <= w_last ? 1u : 0u;
      v0 += on ? p0[k] : 0u;
      v1 += on ? p1[k] : 0u;
      sl += on ? ps[k] : 0u;
    }
  }
  const uint32_t klast = (uint32_t)a.nch * kChunk;
  const uint32_t padfix = (klast - (uint32_t)a.K) * ((uint32_t)rows[0] ^ 0x8080u) + a.bias_k - 32896u * klast;  // see tab_kernel
  v0 -= padfix;
  v1 -= padfix;
  __syncthreads();
  const uint32_t lterm = (uint32_t)a.qd->z_tab * sl;
  const float scale = a.qd->scale;
  const bool wide = a.K > 16384;
  const int i = i0 + 64 * g + 16 * r + m;
  if (i < a.I)
    put_pair<CH>(a, acc_base, y_base, i, j0 + 2 * kg, v0, v1, dequant(v0, lterm, column_constant<4>(cterm, 2 * kg), scale, wide),
                 dequant(v1, lterm, column_constant<4>(cterm, 2 * kg + 1), scale, wide));
}

// ---- operand preparation ---------------------------------------------------------------

// Ready-made tables for tab_kernel<.., PRE>: for every chunk of 16 rows of the packed table-side
// operand and every group g of eight columns the image of one LDS buffer: entry v of tap t,
// (R[b_0][v] .. R[b_7][v]) with b_c = Bp[16 chunk + t][8g + c], at 256 v + 16 t.  One block per image;
// roles as in tab_kernel's own building: lane = (tap, quarter), so that 16 lanes store 256
// contiguous bytes.
__global__ __launch_bounds__(kThreads) void prep_tables_kernel(const uint16_t* __restrict__ rows, const uint8_t* __restrict__ Bp,
                                                               int Jpad, uint8_t* __restrict__ tabs) {
  const int groups = Jpad >> 3;
  const int chunk = blockIdx.x / groups, g = blockIdx.x - chunk * groups;
  const int lane = threadIdx.x & 63, bt = lane & 15, bv = 32 * (threadIdx.x >> 6) + 8 * (lane >> 4);
  const uint2 codes = *reinterpret_cast<const uint2*>(Bp + (size_t)(chunk * kChunk + bt) * Jpad + 8 * g);
  u32x4 d[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t b = ((c < 4 ? codes.x : codes.y) >> (8 * (c & 3))) & 0xffu;
    d[c] = *reinterpret_cast<const u32x4*>(rows + b * 256u + bv);
  }
  uint8_t* image = tabs + (size_t)blockIdx.x * kTabBytes;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    u32x4 v;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      v[c] = __builtin_amdgcn_perm(d[2 * c + 1][e >> 1], d[2 * c][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
    *reinterpret_cast<u32x4*>(image + (bv + e) * 256 + bt * 16) = v;
  }
}

struct ConvView {  // im2col addressing of x
  const uint8_t* x;
  int H, W, Cin, KW, sh, sw, ph, pw, OH, OW, M, K, pad_code;
  const DevQuant* dq;  // non-null: the pad code is the activation zero point held on the device
  int dh, dw;
  uint32_t sx;  // 0x80 for signed codes: every code read or padded is turned into offset binary
};

__device__ __forceinline__ uint32_t pad_of(const ConvView& v) {
  return (((uint32_t)(v.dq ? v.dq->x_zp : v.pad_code)) & 0xffu) ^ v.sx;
}

// rows[t][v] = the product of table-side code t and lane-side code v, both bytes with their top bit
// flipped (the matrix instructions of tab_kernel read them as signed bytes: value - 128).
//
// The same launch packs the table-side operand into Bp[krows][Jpad] (zero fill outside k < K,
// j < J) and sums its columns per segment of `seg_rows` rows: psum[seg][j].  Blocks 0..127 do
// the rows; block 128 + seg * (Jpad/64) + jb does 64 columns of one segment, thread = (4
// columns, one of 16 row phases).
// FROM_X: B[k][j] = im2col(x)[j][k] (lanes are channels) else B[k][j] = w[k*J + j].
// do_rows = 0 leaves the table rows out (the grid then holds the packing blocks only), a grid of
// only the row blocks leaves the packing out, do_qd = 0 leaves the coefficients alone: a layer
// handle prepares what depends on filters and table once and the rest per call.
constexpr int kRowBlocks = 128;
template <bool FROM_X>
__global__ __launch_bounds__(256) void prep_kernel(const uint16_t* __restrict__ lut, uint32_t* __restrict__ rows32,
                                                    const uint8_t* __restrict__ w, ConvView cv, int K, int J, int krows,
                                                    int Jpad, int seg_rows, uint8_t* __restrict__ Bp,
                                                    int32_t* __restrict__ psum, QParams qp, QDev* __restrict__ qd,
                                                    int tables, int do_rows, int do_qd, uint32_t* __restrict__ cnt,
                                                    int ncnt) {
  // arrival counters of tiles that workgroups share (tab_kernel): zero before the first launch
  if (do_qd && blockIdx.x == 0)
    for (int i = threadIdx.x; i < ncnt; i += 256) cnt[i] = 0u;
  if (do_qd && blockIdx.x == 0 && threadIdx.x == 0) {
    int xz = qp.x_zp, wz = qp.w_zp, pad = qp.pad_code;
    float sc = qp.scale;
    if (qp.dq) {
      xz = qp.dq->x_zp;
      wz = qp.dq->w_zp;
      pad = xz;
      sc = qp.dq->x_scale * qp.dq->w_scale;
    }
    // Signed codes c are handled as offset binary c' = c + 128 (their byte with the top bit
    // flipped).  The sums the kernels form are then sums of c', 128 * K too large each, which the
    // constant term takes back: corr = acc - wz*Sp - xz*Sf + K*xz*wz with Sp = Sp' - 128 K etc.
    qd->z_lane = FROM_X ? wz : xz;
    qd->z_tab = FROM_X ? xz : wz;
    qd->kzz = (long long)K * xz * wz + (qp.sgn ? 128LL * K * (xz + wz) : 0LL);
    qd->scale = sc;
    qd->pad4 = (((uint32_t)pad & 0xffu) ^ (qp.sgn ? 0x80u : 0u)) * 0x01010101u;
    for (int e = 0; e < 4; ++e) qd->padrow[e] = qd->pad4;
  }
  const uint32_t sx = qp.sgn ? 0x80u : 0u;  // pattern <-> offset-binary code; also moves int16 entries to offset form
  const int row_blocks = do_rows ? kRowBlocks * tables : 0;
  if ((int)blockIdx.x < row_blocks) {  // kRowBlocks blocks per multiplier table
    const int tbl = blockIdx.x / kRowBlocks;
    lut += (size_t)tbl * 65536;
    rows32 += (size_t)tbl * 32768;
    const int dw = (blockIdx.x - tbl * kRowBlocks) * 256 + threadIdx.x;  // 0 .. 32767
    const int t = dw >> 7, P = dw & 127;
    uint32_t lo, hi;
    const uint32_t tp = (uint32_t)t ^ sx, p0 = (uint32_t)(2 * P) ^ sx, p1 = (uint32_t)(2 * P + 1) ^ sx;
    if (FROM_X) {  // table side = activation code t, lane side = filter code v
      lo = lut[tp * 256 + p0];
      hi = lut[tp * 256 + p1];
    } else {  // table side = filter code t, lane side = activation code v
      lo = lut[p0 * 256 + tp];
      hi = lut[p1 * 256 + tp];
    }
    rows32[dw] = (lo | (hi << 16)) ^ 0x80808080u ^ (sx * 0x01000100u);  // signed entries + 32768
    return;
  }
  __shared__ int32_t red[16][65];
  const int b = blockIdx.x - row_blocks;
  const int jblocks = Jpad / 64;
  const int seg = b / jblocks, jb = b - seg * jblocks;
  const int c4 = threadIdx.x & 15, r = threadIdx.x >> 4;
  const int j = jb * 64 + c4 * 4;
  const int kbeg = seg * seg_rows, kend = min(krows, kbeg + seg_rows);
  const bool fast = !FROM_X && (J % 4 == 0) && (((uintptr_t)w & 3) == 0) && (j + 3 < J);
  int32_t s[4] = {0, 0, 0, 0};
  const uint32_t pad = FROM_X ? pad_of(cv) : 0u;
  int py[4] = {0, 0, 0, 0}, px[4] = {0, 0, 0, 0};  // FROM_X: the column's pixel under tap (0, 0), and its image
  const uint8_t* image[4] = {cv.x, cv.x, cv.x, cv.x};
  if (FROM_X) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ohw = cv.OH * cv.OW, m = min(j + e, J - 1);
      const int n = m / ohw, r = m - n * ohw;
      const int oy = r / cv.OW;
      py[e] = oy * cv.sh - cv.ph;
      px[e] = (r - oy * cv.OW) * cv.sw - cv.pw;
      image[e] = cv.x + (size_t)n * cv.H * cv.W * cv.Cin;
    }
  }
  for (int k = kbeg + r; k < kend; k += 16) {
    uint32_t pk = 0;
    if (k < K) {
      if (fast) {
        pk = *reinterpret_cast<const uint32_t*>(w + (size_t)k * J + j) ^ (sx * 0x01010101u);
      } else {
        int dy = 0, dx = 0, ci = 0;  // FROM_X: the tap (256 patches of 4096: 9.0 us, 9.1 with pixel and tap decoded per byte)
        if (FROM_X) {
          const int tap = k / cv.Cin, ky = tap / cv.KW;
          ci = k - tap * cv.Cin;
          dy = ky * cv.dh;
          dx = (tap - ky * cv.KW) * cv.dw;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t bb = 0;
          if (FROM_X) {
            const int iy = py[e] + dy, ix = px[e] + dx;
            const bool in = (unsigned)iy < (unsigned)cv.H && (unsigned)ix < (unsigned)cv.W;
            if (j + e < J) bb = in ? (uint32_t)image[e][((size_t)iy * cv.W + ix) * cv.Cin + ci] ^ cv.sx : pad;
          } else if (j + e < J) {
            bb = (uint32_t)w[(size_t)k * J + j + e] ^ sx;
          }
          pk |= bb << (8 * e);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += (int32_t)((pk >> (8 * e)) & 0xffu);
    }
    *reinterpret_cast<uint32_t*>(Bp + (size_t)k * Jpad + j) = pk;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) red[r][c4 * 4 + e] = s[e];
  __syncthreads();
  if (threadIdx.x < 64) {
    int32_t t = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) t += red[q][threadIdx.x];
    psum[(size_t)seg * Jpad + jb * 64 + threadIdx.x] = t;
  }
}

// Materialized im2col, Ap[Kp / 16][m][16] (zero fill for k >= K): used when the implicit view cannot be
// read in aligned 16-byte pieces (Cin not a multiple of 16, or a misaligned base pointer).
// Staged form of the same materialization for the usual case (few input channels, e.g. the first layer of a
// network): a block takes r output rows of a stripe of pw output pixels and copies the input rows
// they touch into LDS once (every input byte is used by about KH*KW/(sh*sw) patches).  The stage offsets of
// a chunk's sixteen bytes are the same for every pixel up to the pixel's own offset, so they are decoded
// once per block; a thread then gathers the 16 bytes of one pixel and chunk from LDS and writes them with
// one store, neighbouring threads neighbouring pixels, a wave a contiguous kilobyte.
// Bound: the writes of Ap, beside one LDS read per byte of it.  Blocks of up to 512 pixels, so that the
// round trip of the stage's loads and the decoding are paid seldom: 32 x 32 x 3, 3 x 3, batch 1000 (33 MB
// of patches) 61 us with stripes of 32 pixels and a dword per thread, 17 us now; 224 x 224 x 3, 7 x 7 with
// stride 2, batch 32 (64 MB) 47 us, 28 us now.  Smaller blocks where fewer than
// four per CU would be left (8: 18 and 34 us; 1024 pixels: 22 and 28), narrower ones where fewer than one.
// Where the rows that a block's taps read are fewer than those it spans (dilated filters), they are staged one by one.
struct Im2colTile {
  int pw, r;              // output pixels per row of a block, output rows of a block
  int nstripe, nrows;     // blocks across and down an image
  int npix;               // pw * r
  int row_bytes;          // staged bytes of an input row
  int stage_bytes;        // of the whole stage, a multiple of 16
  // Staged row s is input row first + s: every row that the block spans (group = 0), or only the rows that its taps
  // read, filter row by filter row (GROUPS, group = KH): first + (s / group) * sh + (s % group) * dh.
  int group, spix, stap;  // stage rows per output row, per filter row
  uint32_t pw_mul, npix_mul, row_mul, group_mul;  // floor(i / pw) = umulhi(2 * i, pw_mul), exact for i * pw < 2^31; the others alike
};
template <bool GROUPS>
__global__ __launch_bounds__(256) void prep_im2col_lds_kernel(ConvView cv, int KH, int nch, Im2colTile t,
                                                              uint8_t* __restrict__ Ap) {
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t* stage = smem;                                                 // [input rows][row_bytes]
  uint16_t* offtab = reinterpret_cast<uint16_t*>(smem + t.stage_bytes);  // [nch * 16] stage offsets of a patch's bytes
  const uint32_t pad = pad_of(cv);
  const int n = blockIdx.x / (t.nstripe * t.nrows), rest = blockIdx.x - n * (t.nstripe * t.nrows);
  const int rb = rest / t.nstripe;
  const int oy0 = rb * t.r, ox0 = (rest - rb * t.nstripe) * t.pw;
  const int nr = min(t.r, cv.OH - oy0), npx = min(t.pw, cv.OW - ox0);
  const int ix0 = ox0 * cv.sw - cv.pw, iy0 = oy0 * cv.sh - cv.ph;
  const int total = ((nr - 1) * t.spix + (KH - 1) * t.stap + 1) * t.row_bytes;
  auto input_row = [&](int row) {
    if (!GROUPS) return iy0 + row;
    const int g = (int)__umulhi(2u * (uint32_t)row, t.group_mul);
    return iy0 + g * cv.sh + (row - g * t.group) * cv.dh;
  };
  // Byte b of a staged row is byte ix0 * Cin + b of the input row: in the image for
  // lo_b <= b < hi_b, padding outside.
  const int lo_b = min(max(0, -ix0), t.row_bytes / cv.Cin) * cv.Cin;
  const int hi_b = min(cv.W - ix0, t.row_bytes / cv.Cin) * cv.Cin;
  // Eight bytes per thread at a time, every load unconditional and from an address clamped into the image
  // (what lies outside is replaced afterwards), so that the loads are issued back to back.
  if (hi_b > lo_b) {
    const uint8_t* img = cv.x + (long long)n * cv.H * cv.W * cv.Cin + (long long)ix0 * cv.Cin;
    for (int i0 = threadIdx.x; i0 < total; i0 += 256 * 8) {
      uint32_t v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = min(i0 + 256 * j, total - 1);
        const int row = (int)__umulhi(2u * (uint32_t)i, t.row_mul), b = i - row * t.row_bytes;
        v[j] = img[(long long)min(max(input_row(row), 0), cv.H - 1) * cv.W * cv.Cin + min(max(b, lo_b), hi_b - 1)];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = i0 + 256 * j;
        const int row = (int)__umulhi(2u * (uint32_t)i, t.row_mul), b = i - row * t.row_bytes;
        const bool in = b >= lo_b && b < hi_b && (unsigned)input_row(row) < (unsigned)cv.H;
        if (i < total) stage[i] = (uint8_t)(in ? v[j] ^ cv.sx : pad);
      }
    }
  } else {  // the whole stripe reads padding columns only
    for (int i = threadIdx.x; i < total; i += 256) stage[i] = (uint8_t)pad;
  }
  for (int k = threadIdx.x; k < nch * 16; k += 256) {
    const int tap = k / cv.Cin, ci = k - tap * cv.Cin;
    const int ky = tap / cv.KW, kx = tap - ky * cv.KW;
    offtab[k] = k < cv.K ? (uint16_t)(ky * t.stap * t.row_bytes + kx * cv.dw * cv.Cin + ci) : (uint16_t)0;
  }
  __syncthreads();
  const size_t m0 = ((size_t)n * cv.OH + oy0) * cv.OW + ox0;
  for (int i = threadIdx.x; i < nch * t.npix; i += 256) {
    const int c = (int)__umulhi(2u * (uint32_t)i, t.npix_mul), px = i - c * t.npix;
    const int r = (int)__umulhi(2u * (uint32_t)px, t.pw_mul), ox = px - r * t.pw;
    const bool in = r < nr && ox < npx;
    const uint8_t* from = stage + (in ? r * t.spix * t.row_bytes + ox * cv.sw * cv.Cin : 0);
    const uint4* op = reinterpret_cast<const uint4*>(offtab + c * 16);
    const uint4 oa = op[0], ob = op[1];
    const uint32_t o[8] = {oa.x, oa.y, oa.z, oa.w, ob.x, ob.y, ob.z, ob.w};
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = (uint32_t)from[o[2 * q] & 0xffffu] | (uint32_t)from[o[2 * q] >> 16] << 8 |
             (uint32_t)from[o[2 * q + 1] & 0xffffu] << 16 | (uint32_t)from[o[2 * q + 1] >> 16] << 24;
    const int left = cv.K - c * 16;  // bytes of this chunk that belong to the patch
    if (left < 16) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] &= left >= 4 * q + 4 ? ~0u : left <= 4 * q ? 0u : (1u << (8 * (left - 4 * q))) - 1u;
    }
    if (in)
      *reinterpret_cast<uint4*>(Ap + ((size_t)c * (size_t)cv.M + m0 + (size_t)r * cv.OW + ox) * 16) =
          make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// One thread per 16-byte piece: the pixel is decoded once and the tap index advanced
// incrementally; consecutive threads take consecutive pixels of one chunk and so write
// consecutive pieces of the chunk-major Ap.
__global__ __launch_bounds__(256) void prep_im2col_kernel(ConvView cv, int Kp, uint8_t* __restrict__ Ap) {
  const uint32_t nchunk = (uint32_t)Kp / 16u;
  const uint32_t q = blockIdx.x * 256u + threadIdx.x;
  if (q >= (uint32_t)cv.M * nchunk) return;  // M * Kp/16 < 2^31: see tab_supported
  const uint32_t chunk = q / (uint32_t)cv.M;
  const uint32_t m = q - chunk * (uint32_t)cv.M;
  const int k0 = (int)chunk * 16;
  const uint32_t ohw = (uint32_t)(cv.OH * cv.OW);
  const uint32_t n = m / ohw, r = m - n * ohw;
  const int oy = (int)(r / (uint32_t)cv.OW), ox = (int)(r - (r / (uint32_t)cv.OW) * (uint32_t)cv.OW);
  const int by = oy * cv.sh - cv.ph, bx = ox * cv.sw - cv.pw;
  int tap = k0 / cv.Cin, ci = k0 - tap * cv.Cin;
  int ky = tap / cv.KW, kx = tap - ky * cv.KW;
  uint32_t pk[4] = {0, 0, 0, 0};
  const uint32_t pad = pad_of(cv);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if (k0 + e < cv.K) {
      const int iy = by + ky * cv.dh, ix = bx + kx * cv.dw;
      uint32_t v = pad;
      if ((unsigned)iy < (unsigned)cv.H && (unsigned)ix < (unsigned)cv.W)
        v = (uint32_t)cv.x[((size_t)(n * cv.H + iy) * cv.W + ix) * cv.Cin + ci] ^ cv.sx;
      pk[e >> 2] |= v << (8 * (e & 3));
      if (++ci == cv.Cin) {
        ci = 0;
        if (++kx == cv.KW) { kx = 0; ++ky; }
      }
    }
  }
  *reinterpret_cast<uint4*>(Ap + ((size_t)chunk * (size_t)cv.M + m) * 16) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
}

// Activations chunk by chunk, out[C / 16][P][16]: position p = (n, oy, ox) is pixel (n, oy*sh - ph,
// ox*sw - pw) of x, or the pad code outside the image: strides 1 copy the tensor, with the border
// that ph and pw give it.  A wave of tab_kernel reads 16 channels of 64 consecutive pixels at a time:
// from this layout one contiguous kilobyte, where the tensor as it stands costs a 128-byte line per
// pixel and chunk, and with the border no tap lies outside.  Signed codes are turned into offset
// binary on the way (sx4).  A block turns 512 pieces of 16 bytes through LDS: 2^cl chunks (up to 8 =
// 128 channels) of 512 >> cl positions.  Bound by memory: 16 channels of a million pixels with border
// (35 MB) take 7 us, 23 with eight chunks per block whatever the channel count.
__global__ __launch_bounds__(256) void prep_chunks_kernel(const uint8_t* __restrict__ x, int P, int C, int cl, int H, int W,
                                                          int OHW, int OW, int sh, int sw, int ph, int pw, uint32_t sx4,
                                                          const QDev* __restrict__ qd, uint8_t* __restrict__ out) {
  __shared__ uint4 tile[512 + 8];
  const int pl = 9 - cl, np = 1 << pl;  // positions of a block
  const int p0 = blockIdx.x * np, ck0 = blockIdx.y << cl, nck = min(1 << cl, C / 16 - ck0);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = threadIdx.x + 256 * h, ck = q & ((1 << cl) - 1), pos = q >> cl, p = p0 + pos;
    if (ck < nck && p < P) {
      const int n = p / OHW, r = p - n * OHW;
      const int oy = r / OW;
      const int iy = oy * sh - ph, ix = (r - oy * OW) * sw - pw;
      uint4 v;
      if ((unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W) {
        v = *reinterpret_cast<const uint4*>(x + ((size_t)(n * H + iy) * W + ix) * C + (size_t)(ck0 + ck) * 16);
        v.x ^= sx4; v.y ^= sx4; v.z ^= sx4; v.w ^= sx4;
      } else {
        v = *reinterpret_cast<const uint4*>(qd->padrow);
      }
      tile[ck * (np + 1) + pos] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = threadIdx.x + 256 * h, ck = q >> pl, pos = q & (np - 1), p = p0 + pos;
    if (ck < nck && p < P) *reinterpret_cast<uint4*>(out + ((size_t)(ck0 + ck) * P + p) * 16) = tile[ck * (np + 1) + pos];
  }
}

// Ap[k / 16][j][k % 16] = w[k][j] (zero fill for k >= K).  A thread takes one chunk of sixteen rows and four
// neighbouring columns: a dword per row, all in flight together, turned in registers (4 x 4 bytes in eight permutes),
// and four 16-byte pieces.  Rows may start at any byte (dwords at their own alignment); for columns past the last whole four
// the dword of the last four is moved down (read byte by byte, row after row, the one such thread kept its wave waiting:
// 122 x 60 x 2819 22.9 us the call, 20.5 so).  Bound by memory: 4096 x 4096 (34 MB) 35 us with byte loads and a pass
// through LDS, 10 us now.
__global__ __launch_bounds__(256) void prep_transpose_kernel(const uint8_t* __restrict__ w, int K, int J,
                                                              uint8_t* __restrict__ Ap, uint32_t sx) {
  const int chunk = blockIdx.x, j = 4 * (blockIdx.y * 256 + threadIdx.x);
  if (j >= J) return;
  const int k0 = chunk * kChunk, nk = min(kChunk, K - k0);
  const int jb = min(j, max(J - 4, 0)), late = J < 4 ? 0 : 8 * (j - jb);  // past the last whole four: the last four columns, moved down
  uint32_t v[kChunk];  // columns j .. j + 3 of a row; past the last row: that one again, cleared below
  if (J >= 4) {
#pragma unroll
    for (int e = 0; e < kChunk; ++e) v[e] = load_any<uint32_t>(w + (size_t)(k0 + min(e, nk - 1)) * J + jb);
  } else {
#pragma unroll
    for (int e = 0; e < kChunk; ++e) {
      const uint8_t* row = w + (size_t)(k0 + min(e, nk - 1)) * J;
      v[e] = row[0] | (uint32_t)row[min(1, J - 1)] << 8 | (uint32_t)row[min(2, J - 1)] << 16;
    }
  }
  uint32_t piece[4][4];  // [column][four rows]
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = 4 * q + e < nk ? (v[4 * q + e] >> late) ^ (sx * 0x01010101u) : 0u;
    const uint32_t lo01 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
    piece[0][q] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    piece[1][q] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    piece[2][q] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    piece[3][q] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
  uint4* out = reinterpret_cast<uint4*>(Ap) + (size_t)chunk * J + j;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (j + c < J) out[c] = make_uint4(piece[c][0], piece[c][1], piece[c][2], piece[c][3]);
}

// ---- host side -------------------------------------------------------------------------

static inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// What the byte loads of prep_im2col_kernel cost: a wave takes one chunk of taps of neighbouring pixels.
struct PatchLines {
  double inside, u, far;  // share of taps inside the image, bytes between neighbouring pixels / 128 (1 at most), 0 .. 1: the images beyond the L2s
  PatchLines(const ConvView& cv, int KH, int N) {
    const double span_h = (double)(cv.OH - 1) * cv.sh + (double)(KH - 1) * cv.dh + 1.0;
    const double span_w = (double)(cv.OW - 1) * cv.sw + (double)(cv.KW - 1) * cv.dw + 1.0;
    const double xbytes = (double)N * cv.H * cv.W * cv.Cin, pixels = (double)N * cv.OH * cv.OW;
    inside = std::min(1.0, cv.H / span_h) * std::min(1.0, cv.W / span_w);
    u = std::min(1.0, std::max((double)cv.Cin * cv.sw, xbytes / pixels) / 128.0);
    far = std::min(1.0, std::max(0.0, xbytes / 8e6 - 1.0));
  }
};
// Its time, seconds: 8 ps per 16-byte piece where pixels share lines, 50 where they do not, 60 to 220 where the images do not
// fit the L2s either, since every chunk of taps walks through all of them (1800 random layers; the last scatter with the
// XCDs that the blocks of a chunk fall on and count 100).
static double general_copy(const ConvView& cv, int KH, int N, int nch) {
  const PatchLines l(cv, KH, N);
  const double far = std::min(1.0, std::max(0.0, (double)N * cv.H * cv.W * cv.Cin / 12e6 - 1.0));
  return (double)N * cv.OH * cv.OW * nch * (8e-12 + l.inside * (42e-12 * l.u * l.u + (l.u == 1.0 ? 50e-12 * far : 0.0)));
}

// False: prep_im2col_kernel, where the stage cannot hold a block or is the slower form.  Staged, a block takes 1.5 ns of
// the machine and 1.15 ps per staged byte.  The other form is priced at 5.7 ps per 16-byte piece and up to 36 to 89 ps for the
// lines that its loads touch (less than the medians of general_copy, which scatter by a factor of two and more).
// Fitted to 3400 random layers (1 to 300000 images, dilations, strides): the rule's sum of times is 1 % above that of the
// better form each time and 26 layers are on one that is more than 20 % slower; always staged 15 % above, never 186 %.
// Many small images are the case where it matters (120191 of 4 x 4 x 4, 2 x 1 filter: staged 143 us, 19 otherwise).
static bool im2col_tile(const ConvView& cv, int KH, int N, int Kp, Im2colTile* t) {
  if (Kp > 4096) return false;
  const int nch = Kp / 16;
  auto row_bytes = [&](int pw) { return ((long long)(pw - 1) * cv.sw + (long long)(cv.KW - 1) * cv.dw + 1) * cv.Cin; };
  // staged rows for r output rows: all that they span, or their taps' rows one by one
  auto spanned = [&](int r) { return (long long)(r - 1) * cv.sh + (long long)(KH - 1) * cv.dh + 1; };
  auto rows = [&](int r) { return std::min(spanned(r), (long long)r * KH); };
  int pw = cdiv(cv.OW, cdiv(cv.OW, 256));
  while (row_bytes(pw) * rows(1) > 32768 && pw > 1) pw = cdiv(pw, 2);
  while ((long long)N * cv.OH * cdiv(cv.OW, pw) < 256 && cdiv(pw, 2) * nch >= 64 && pw > 1) pw = cdiv(pw, 2);
  const long long rb = row_bytes(pw);
  if (rb * rows(1) > 32768) return false;
  const int nstripe = cdiv(cv.OW, pw);
  int r = 1;
  while (r < cv.OH && pw * (r + 1) <= 512 && rb * rows(r + 1) <= 16384 && (long long)N * nstripe * cdiv(cv.OH, r + 1) >= 1024) ++r;
  const long long blocks = (long long)N * nstripe * cdiv(cv.OH, r), bytes = rb * rows(r);
  if (blocks >= (1LL << 24)) return false;  // a launch holds fewer than 2^32 threads
  const PatchLines l(cv, KH, N);
  const double general = (double)N * cv.OH * cv.OW * nch *
                         (0.0057 + (0.036 + 0.023 * l.far) * std::sqrt(l.inside) * l.u + (l.u == 1.0 ? 0.03 * l.far * l.inside : 0.0));
  if (blocks * (1.5 + 1.15e-3 * bytes) > general + 500.0) return false;  // ns; half a microsecond decides nothing
  const bool taps = rows(r) < spanned(r);
  auto mul = [](int d) { return (uint32_t)(((1ull << 31) + d - 1) / d); };
  const int stage = (int)((bytes + 15) & ~15ll);
  *t = {pw, r, nstripe, cdiv(cv.OH, r), pw * r, (int)rb, stage, taps ? KH : 0, taps ? KH : cv.sh, taps ? 1 : cv.dh,
        mul(pw), mul(pw * r), mul((int)rb), mul(KH)};
  return true;
}
// 1 x 1 filters that read every pixel: the images as one row of pixels.
static void im2col_flatten(ConvView* cv, int KH, int* N) {
  if (KH != 1 || cv->KW != 1 || cv->ph || cv->pw || cv->sh != 1 || cv->sw != 1) return;
  if (cv->OH != cv->H || cv->OW != cv->W) return;
  cv->W = cv->OW = cv->M;
  cv->H = cv->OH = *N = 1;
}

// Tile configurations: the greatest height of a tile in lane elements (tiles are 8 columns wide).  The
// "tile" option selects one by index + 1; the automatic choice is the full height of the kernel.
static const int kTiles[] = {512, 1024, kIT, 1536, 2048, 2560, 3072};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int kFullTile = 2;
int tab_num_tiles() { return kNumTiles; }

bool reads_in_place(const Geom& g, const void* x) { return g.Cin % 16 == 0 && ((uintptr_t)x & 15) == 0; }

// The preparation kernels index their pieces with 32-bit integers.
bool tab_supported(const Geom& g) {
  if (g.mult || g.groups > 1) return false;  // depthwise: every output channel has its own lane-side operand;
                                              // grouped: the channel blocks would each need strided views
  const long long chunks = cdiv(g.K, kChunk);
  // tile indices over all tables and the fix-up grid are 32-bit: tiles hold at least 64 x 8 outputs
  if ((double)g.M * g.Cout * g.T >= 5.0e10) return false;
  return (long long)g.M * chunks < (1LL << 31) && (long long)g.Cout * chunks < (1LL << 31);
}

int cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    n = (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess &&
         prop.multiProcessorCount > 0)
            ? prop.multiProcessorCount
            : 256;
  }
  return n;
}

// Number of partial tile pieces that a grid of G workgroups produces (see tab_kernel); the
// largest number of pieces that one tile is cut into and of segments that one workgroup runs.
// Walks the shares by addition (position = tile, chunk of it): it is asked for dozens of grids per layer.
static int count_partials(int ntiles, int nch, int G, int* most_per_tile, int* most_segs) {
  const long long total = (long long)ntiles * nch;
  const long long share = total / G, rest = total % G;
  const int step_t = (int)(share / nch), step_c = (int)(share % nch);
  int n = 0, most = 0, run = 0, segs = 0, t = 0, c = 0, run_tile = -1;
  long long carry = 0;
  auto piece = [&](int tile) {
    ++n;
    run = tile == run_tile ? run + 1 : 1;
    run_tile = tile;
    most = std::max(most, run);
  };
  for (int w = 0; w < G; ++w) {
    int t1 = t + step_t, c1 = c + step_c;  // end of the share
    if ((carry += rest) >= G) { carry -= G; ++c1; }
    if (c1 >= nch) { c1 -= nch; ++t1; }
    if (t1 == t) {  // within one tile
      if (c1 > c) { segs = std::max(segs, 1); piece(t); }
    } else {
      segs = std::max(segs, t1 - t + (c1 ? 1 : 0));
      if (c) piece(t);
      if (c1) piece(t1);
    }
    t = t1;
    c = c1;
  }
  *most_per_tile = most;
  *most_segs = segs;
  return n;
}

// Cost model of one (tile height, lane assignment, grid size) choice, in seconds; measured on dense and
// convolution layers with the heights, cuts and combinations forced.
//   - a phase (a chunk of 16 taps) of a tile of ih lane elements: 1.2 us for its tables, barrier
//     and latencies (1.05 us with ready-made tables) and 0.6 ns per lane element;
//   - every segment a workgroup runs: its first tables, the pipeline fill and its stores.
//     Both are prices of earlier forms of the kernel (a phase is a fifth to an eighth shorter now and the ready-made
//     one is the longer one on low tiles, see assembled_gain; a segment takes 3 us less).  They are used for the order of
//     grids and heights and for the comparison with fewpix_kernel, which is fitted to them as they are;
//   - tiles cut into pieces: a launch of the fix-up kernel and the pieces once written and once read,
//     or, combined inside the main kernel, the reading of the others' pieces one after another;
//   - grids larger than the machine run in rounds.
//   - the lane dimension may be cut into more (lower) tiles than it needs, when that makes the
//     tile count fill whole rounds of the machine, or whole multiples of it with K slices.
struct PlanChoice { int tile, variant, G, partials, nti, ih; double cost; int most; };
// Pieces are combined inside tab_kernel by the workgroup that finishes last where it has to read at
// most kCombineElems lane elements of the others (177 random layers 0.98 of the time with the second launch), and up to
// kCombineMost pieces of sums of at least kCombineLong chunks (two or three pieces 0.99; 28 x 28 x 128 3 x 3 at batch 32, two pieces of
// 3136 x 8: 130.2 us, 137.4 with the second launch).  Others go through tab_fixup_kernel, which spreads the sums of one
// tile over many blocks: four pieces of long sums 0.96 (14 x 14 x 1024 1 x 1 to 256 at batch 32, four of 3136: 72.5 us, 89.3
// in the kernel; 7 x 7 x 512 3 x 3, four of 1600: 148.2 and 152.5), where all workgroups end at once and a quarter
// of them is left with the work.
constexpr int kCombineElems = 768, kCombineMost = 3, kCombineLong = 64;
// Ready-made tables that a layer gets without being asked to: any set of up to kPreTablesSmall
// bytes (it stays in the L2s and the memory-side cache whichever workgroup reads which part:
// the CIFAR-shaped layers with K slices gain 25 %), larger sets (up to kPreTablesMax bytes) for
// layers with at least kPreRowTiles tiles along the lanes and no K slices.
constexpr size_t kPreTablesSmall = (size_t)20 << 20;
constexpr size_t kPreTablesMax = (size_t)32 << 20;
constexpr int kPreRowTiles = 8;

// Pieces are combined by the main kernel (see kCombineElems).
static bool combines(const Options& o, int partials, int most, int ih, int nch) {
  if (partials == 0) return false;
  if (o.combine) return o.combine == 2;
  return (long long)(most - 1) * ih <= kCombineElems || (most <= kCombineMost && nch >= kCombineLong);
}
// Ready-made tables (one 4 KiB table per tap and group of eight columns) where the filters are
// the table side and one multiplier table is used.  Every workgroup reads the tables of its taps
// and columns from global memory, so they pay where many tiles along the lane dimension read the
// same tables at about the same time (the reads then meet in the L2s) or where all of them stay in
// the caches.
static size_t table_bytes(const Geom& g) {
  return ((size_t)cdiv(g.K, kChunk) * kChunk + 1) * ((size_t)cdiv(g.Cout, 64) * 64 / 8) * 4096;
}
static bool ready_made(const Geom& g, const Options& o, int v, int partials, int nti) {
  const size_t bytes = table_bytes(g);
  if (v != 2 || g.T != 1 || bytes > ((size_t)1 << 30)) return false;
  if (o.tables) return o.tables == 2;
  return bytes <= kPreTablesSmall || (partials == 0 && nti >= kPreRowTiles && bytes <= kPreTablesMax);
}

// What a share of `iters` chunks in `segs` segments of ih lane elements (at most half the full height) gains, us, with tables
// assembled in the kernel instead of ready-made ones, for the layers that give those up.  misses: the share of its table copies
// that no other workgroup of the XCD has fetched, 0 for sets that stay in the L2s anyway.  Fitted to 1533 random layers, each
// timed in both forms back to back and with 48 MB read and written in between (misses by 0.7 us rms): a phase is 0.24 us shorter
// assembled, less 0.16 per 1024 elements, and another 0.70, less 0.18 per 1024, where ready-made tables come from beyond the
// L2; a segment's first tables take two round trips to memory instead of one, 2 us more (1.4 from beyond the L2).
// Prepared layers give their tables up for more than 0.5 us: of 2200 layers they then take 0.987 of the time with all tables
// ready-made (cold 0.993), 10 are more than 3 % slower so and 2 more than 8 %.  From phases and segments measured one by one,
// without regard to who shares the tables, shares of one to three chunks were given up as well (63 and 41 layers slower; 852 x 32 x
// 869, two chunks: 15.2 us, 13.6 ready-made).  1113 x 78 x 379: 22.7 us ready-made, 17.7 assembled.  Where a second launch sums the
// pieces the fit is worse and the line 1.5 us (128 x 8 x 8 x 64, 3 x 3 to 64: 37.3 us ready-made, 34.4 assembled, every
// copy a miss; 3 x 28 x 28 x 64, one in four: 20.0 and 21.9).
// Calls that prepare their constants spend 7 us and more on the tables (choose_route) and keep them for more than 3 us.
// Not asked for tiles above half the height, where neither form is ahead by much (assembled -5 to +6 % of a launch).
static double assembled_gain(int ih, long long iters, int segs, double misses) {
  return iters * (0.24 - 0.16e-3 * ih + misses * (0.70 - 0.18e-3 * ih)) - segs * (2.0 - 0.6 * misses);
}

static PlanChoice plan_choice_nti(const Geom& g, const Options& o, int tile, int v, int nti_wanted) {
  const long long I = (v == 2) ? g.M : g.Cout;
  const long long J = (v == 2) ? g.Cout : g.M;
  // balanced tile height (padding spread over all tiles, in steps of one wave), then as many
  // tiles as that height needs (rounding the height up can free the last one)
  const int ih = cdiv(cdiv(I, nti_wanted), 64) * 64;
  const int nti = cdiv(I, ih);
  const int ntiles = nti * cdiv(J, kJT) * g.T;
  const int nch = cdiv(g.K, kChunk);
  const long long total = (long long)ntiles * nch;
  const int slots = cu_count();
  auto evaluate = [&](int Gc) {
    PlanChoice c{tile, v, Gc, 0, nti, ih, 0.0, 0};
    int segs = 1;
    c.partials = count_partials(ntiles, nch, Gc, &c.most, &segs);
    const double t_chunk = (ready_made(g, o, v, c.partials, nti) ? 1.05e-6 : 1.2e-6) + 0.6e-9 * ih;
    const double t_seg = 2.5e-6 + 1.6e-9 * ih;
    const double rounds = std::ceil((double)Gc / slots);
    const double iters = std::ceil((double)total / Gc);
    c.cost = rounds * (iters * t_chunk + segs * t_seg);
    // four pieces of a long sum are priced like three: priced by their bytes, grids of three or fewer pieces are taken instead,
    // which are slower (100 random layers 1.01)
    if (combines(o, c.partials, c.most, ih, nch) || (c.partials && !o.combine && c.most == kCombineMost + 1 && nch >= kCombineLong))
      c.cost += 2.32e-6 + (c.most - 1) * 0.5e-9 * ih;
    else if (c.partials)
      c.cost += 5e-6 + c.partials * 2.0 * ih * kJT * 4.0 / 4.0e12;
    return c;
  };
  if (o.split_k > 0)
    return evaluate((int)std::max<long long>(1, std::min<long long>(std::min<long long>(total, 4LL * slots), (long long)ntiles * o.split_k)));
  // A workgroup per tile, or the fewest whole tiles per workgroup that a launch (fewer than 2^32 threads) holds.
  constexpr int kMostGroups = (int)((1LL << 32) / kThreads) - 1;
  int whole = ntiles;
  for (int d = ntiles / kMostGroups + 1; whole > kMostGroups; ++d) {
    if (d > 4096) whole = slots;
    else if (ntiles % d == 0) whole = ntiles / d;
  }
  PlanChoice best = evaluate(whole);
  std::vector<int> cand;
  if (total >= 2) cand.push_back((int)std::min<long long>(slots, total / 2));
  for (int sdiv = 2; sdiv <= 16; ++sdiv)
    if ((long long)ntiles * sdiv <= slots && nch / sdiv >= 2) cand.push_back(ntiles * sdiv);
  for (int Gc : cand) {
    if (Gc < 1) continue;
    const PlanChoice c = evaluate(Gc);
    // Fewer workgroups than tiles only to cut tiles: with whole tiles a workgroup would go from column to column of one
    // row of tiles, and the 32 bytes that each column has of a line of the output would leave the L2 one by one
    // (38628 x 6 x 208, 18 tables: 470 us, 340 with a workgroup per tile; 1444000 x 16 x 20: 87 and 73).
    if (c.partials == 0 && Gc < ntiles) continue;
    if (c.cost < best.cost) best = c;
  }
  return best;
}

static PlanChoice plan_choice(const Geom& g, const Options& o, int tile, int v) {
  const long long I = (v == 2) ? g.M : g.Cout;
  const long long J = (v == 2) ? g.Cout : g.M;
  const int base = cdiv(I, kTiles[tile]), ntj = cdiv(J, kJT) * g.T;  // column tiles of all tables
  const int most = (int)std::min<long long>(cdiv(I, 64), 8LL * base + 1);
  if (o.row_tiles > 0) return plan_choice_nti(g, o, tile, v, std::max(base, std::min(o.row_tiles, cdiv(I, 64))));
  PlanChoice best = plan_choice_nti(g, o, tile, v, base);
  if (o.split_k > 0) return best;
  // more, lower tiles: those that make 1 .. 4 rounds of the machine, or a half, a third .. an
  // eighth of one for K slices
  const int slots = cu_count();
  int tried = base;
  auto attempt = [&](long long n) {
    if (n <= base || n > most || n == tried) return;
    tried = (int)n;
    const PlanChoice c = plan_choice_nti(g, o, tile, v, (int)n);
    if (c.cost < best.cost) best = c;
  };
  for (int r = 1; r <= 4; ++r) attempt((long long)r * slots / ntj);
  for (int r = 2; r <= 8; ++r) attempt(slots / ((long long)r * ntj));
  attempt(most);
  return best;
}

static TabPlan tab_plan_uncached(const Geom& g, const Options& o, bool prepared);

// Operand bytes that the eight L2s fetch in total when share w of G (iterations w*total/G ..) runs
// on XCD w % 8 (xcd = 0) or when the shares are dealt out XCD by XCD (xcd = 1): per XCD the
// distinct (lane tile, chunk) and (column tile, chunk) pairs its shares touch.  The tables of a
// multi-table call share both operands.  table_copies: how many (column tile, chunk) pairs of these there are.
constexpr long long kMostWalked = 1LL << 22;  // iteration spaces beyond are not worth walking
static double xcd_fetch_bytes(int xcd, int G, int nti, int ntj, int nch, int T, int ih, int jt, long long* table_copies = nullptr) {
  const long long total = (long long)nti * ntj * nch * T;
  const int words = (nch + 63) / 64;  // a bit per chunk
  std::vector<uint64_t> seen_a((size_t)nti * words), seen_b((size_t)ntj * words);
  auto mark = [&](uint64_t* seen, int c0, int c1) {  // chunks c0 .. c1 - 1; returns how many are new
    int fresh = 0;
    for (int k = c0 / 64; k <= (c1 - 1) / 64; ++k) {
      uint64_t m = ~0ull;
      if (k == c0 / 64) m &= ~0ull << (c0 & 63);
      if (k == (c1 - 1) / 64) m &= ~0ull >> (63 - ((c1 - 1) & 63));
      fresh += __builtin_popcountll(m & ~seen[k]);
      seen[k] |= m;
    }
    return fresh;
  };
  const int q = G >> 3, r = G & 7;
  double bytes = 0.0;
  for (int x = 0; x < 8; ++x) {
    std::fill(seen_a.begin(), seen_a.end(), 0);
    std::fill(seen_b.begin(), seen_b.end(), 0);
    long long na = 0, nb = 0;
    const int w0 = xcd ? x * q + std::min(x, r) : x;
    const int nw = q + (x < r ? 1 : 0);
    for (int k = 0; k < nw; ++k) {
      const int w = xcd ? w0 + k : x + 8 * k;
      long long it = (long long)w * total / G;
      const long long e = (long long)(w + 1) * total / G;
      while (it < e) {
        const long long gt = it / nch;
        const int c0 = (int)(it - gt * nch), c1 = (int)std::min<long long>(nch, c0 + (e - it));
        const int tile = (int)(gt % ((long long)nti * ntj));
        const int ti = tile / ntj, tj = tile - ti * ntj;
        na += mark(&seen_a[(size_t)ti * words], c0, c1);
        nb += mark(&seen_b[(size_t)tj * words], c0, c1);
        it += c1 - c0;
      }
    }
    bytes += 16.0 * ((double)na * ih + (double)nb * jt);
    if (table_copies) *table_copies += nb;
  }
  return bytes;
}

// Planning walks over candidate grids and counts their partial pieces, which takes tens of
// microseconds: as much as a small layer's kernels.  Plans are therefore remembered per
// (geometry, options, whether constants are prepared beforehand); the table is small and cleared when it grows past a bound.
TabPlan tab_plan(const Geom& g, const Options& o, bool prepared) {
  struct Key {
    int v[25];
    bool operator<(const Key& other) const { return std::memcmp(v, other.v, sizeof(v)) < 0; }
  };
  static std::mutex mu;
  static std::map<Key, TabPlan> cache;
  const Key k{{g.N, g.H, g.W, g.Cin, g.KH, g.KW, g.Cout, g.sh, g.sw, g.ph, g.pw, g.dh, g.dw, g.sgn, g.mult, o.variant,
               o.split_k, o.tile, o.row_tiles, cu_count(), g.T, o.share_order, o.combine, o.tables, prepared}};
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(k);
  if (it != cache.end()) return it->second;
  if (cache.size() > 4096) cache.clear();
  const TabPlan p = tab_plan_uncached(g, o, prepared);
  cache.emplace(k, p);
  return p;
}

static TabPlan tab_plan_uncached(const Geom& g, const Options& o, bool prepared) {
  TabPlan p{};
  // Lane assignment and tiles: the cheaper by the cost model, with what a call does around the main kernel
  // (launches, the copy or patch matrix of the activations for pixel lanes, the packed patches for
  // channel lanes): over the ResNet-50 layers at batch 1 to 4 and dense layers a run takes the model's
  // time plus 3 to 8 us (activations read 16 channels at a time), plus 9 and 0.8 us a megabyte (patch
  // matrix; without a staged form its own price) or plus 7 to 12 (channel lanes).
  const double xbytes = (double)g.M * g.K;
  ConvView rows{nullptr, g.H, g.W, g.Cin, g.KW, g.sh, g.sw, g.ph, g.pw, g.OH, g.OW, g.M, g.K, 0, nullptr, g.dh, g.dw, 0};
  int images = g.N;
  im2col_flatten(&rows, g.KH, &images);
  Im2colTile stripe;
  const bool staged = im2col_tile(rows, g.KH, images, cdiv(g.K, kChunk) * kChunk, &stripe);
  const double around[2] = {g.Cin % 16 == 0 ? 6e-6 : 9e-6 + (staged ? 0.8e-12 * xbytes : general_copy(rows, g.KH, images, cdiv(g.K, kChunk))),
                            9.1e-6 + 5e-12 * xbytes};
  PlanChoice best{0, 0, 0, 0, 0, 0, 1e30, 0};
  for (int v = 2; v <= 3; ++v) {
    if ((o.variant == 2 || o.variant == 3) && v != o.variant) continue;
    PlanChoice c = plan_choice(g, o, o.tile >= 1 ? o.tile - 1 : kFullTile, v);
    c.cost += around[v - 2];
    if (c.cost < best.cost) best = c;
  }
  const int v = best.variant;
  p.cost = best.cost;
  p.variant = best.variant;
  p.tile = best.tile;
  p.G = best.G;
  p.partials = best.partials;
  p.combine = combines(o, best.partials, best.most, best.ih, cdiv(g.K, kChunk)) ? 1 : 0;
  p.nti = best.nti;
  p.ih = best.ih;
  {
    // numbering of the shares: whichever lets the XCDs' L2s fetch less (ties and very large
    // iteration spaces, not worth walking: XCD by XCD)
    const int ntj = cdiv((v == 2) ? g.Cout : g.M, kJT), nchk = cdiv(g.K, kChunk);
    p.xcd = 1;
    if (o.share_order) {
      p.xcd = o.share_order - 1;
    } else if ((long long)p.nti * ntj * nchk * g.T <= kMostWalked && best.G >= 16) {
      const double f1 = xcd_fetch_bytes(1, best.G, p.nti, ntj, nchk, g.T, p.ih, kJT);
      const double f0 = xcd_fetch_bytes(0, best.G, p.nti, ntj, nchk, g.T, p.ih, kJT);
      if (f0 < 0.9 * f1) p.xcd = 0;
    }
  }
  const int G = best.G;
  const long long I = (v == 2) ? g.M : g.Cout;
  const long long J = (v == 2) ? g.Cout : g.M;
  const int nch = cdiv(g.K, kChunk);

  const size_t Kp = (size_t)nch * kChunk;
  const size_t Jpad = (size_t)cdiv(J, 64) * 64;
  // Prepared block: what depends on filters, table and coefficients.  Scratch block: what depends
  // on the activations.  The packed table-side operand is the filters for pixel lanes and the
  // transposed patch matrix for channel lanes; the materialized lane-side operand the other way round.
  const size_t bpack = up256((Kp + 1) * Jpad), bsum = up256(Jpad * 4 * kMaxSeg);
  // materialized lane operand, or (signed codes, implicit patch view) the offset-binary copy of x
  const size_t apack = up256(std::max((size_t)I * Kp, v == 2 ? (size_t)g.N * g.H * g.W * g.Cin : (size_t)0));
  size_t prep = 0, ws = 0;
  p.off_rows = prep;  prep += up256((size_t)131072 * g.T);
  p.off_qd = prep;    prep += 256;
  p.off_cnt = prep;
  if (p.combine) prep += up256((size_t)p.nti * cdiv(J, kJT) * g.T * 4);
  const size_t tabs_bytes = table_bytes(g);
  p.pre = p.may_pre = ready_made(g, o, v, best.partials, best.nti) ? 1 : 0;
  if (p.pre && !o.tables && best.ih <= kIT / 2) {
    const int ntj = cdiv(J, kJT);
    const long long iters = (long long)best.nti * ntj * nch;
    const double far = std::min(1.0, std::max(0.0, ((double)nch * ntj * kTabBytes - 2e6) / 4e6));  // 0: in the L2s, 1: not
    long long copies = 0;
    if (far > 0.0 && iters <= kMostWalked) xcd_fetch_bytes(p.xcd, best.G, p.nti, ntj, nch, 1, p.ih, kJT, &copies);
    int most, segs;
    count_partials(best.nti * ntj, nch, best.G, &most, &segs);
    const double gain = assembled_gain(best.ih, cdiv(iters, best.G), segs, far * copies / iters);
    if (gain > (!prepared ? -3.0 : best.partials && !p.combine ? 1.5 : 0.5)) p.pre = 0;
  }
  p.off_tabs = prep;
  if (p.pre) prep += up256(tabs_bytes);
  if (v == 2) {
    p.off_bpack = prep;  prep += bpack;
    p.off_bsum = prep;   prep += bsum;
  } else {
    p.off_apack = prep;  prep += apack;
    p.off_bpack = ws;    ws += bpack;
    p.off_bsum = ws;     ws += bsum;
  }
  p.off_lsum = ws;
  p.off_part = ws;
  if (p.partials) {  // two slots per workgroup, each one tile high
    ws += up256((size_t)2 * G * p.ih * 4);
    p.off_part = ws;
    ws += up256((size_t)2 * G * p.ih * kJT * 4);
  }
  // last, so that a call whose activations can be read in place needs the scratch only up to here
  p.ws_apack = 0;
  if (v == 2) {
    p.off_apack = ws;
    p.ws_apack = apack;
    ws += apack;
  }
  p.prep_total = prep;
  p.ws_total = ws;
  return p;
}

// First error of a sequence of launches: every launch is followed by a look at the runtime's
// error state, and nothing more is enqueued after a failure.
#define AX_LAUNCHED()                               \
  do {                                              \
    const hipError_t e_ = hipGetLastError();        \
    if (e_ != hipSuccess) return e_;                \
  } while (0)

// phases: kPhMain and / or kPhFixup (the latter only for plans with partial pieces)
template <int GR, bool CH>
static void launch_tab_kernel(const TabArgs& a, int G, hipStream_t s) {
  void (*k)(TabArgs) = CH                      ? tab_kernel<GR, true, false, false>  // the lane side is the transposed filters
                       : a.tabs && a.padded    ? tab_kernel<GR, false, true, true>
                       : a.tabs                ? tab_kernel<GR, false, true, false>
                       : a.padded              ? tab_kernel<GR, false, false, true>
                                               : tab_kernel<GR, false, false, false>;
  hipLaunchKernelGGL(k, dim3(G), dim3(kThreads), 0, s, a);
}
template <bool CH>
static hipError_t launch_main(const TabArgs& a, int G, int ntiles, int phases, int reps, hipStream_t s) {
  for (int r = 0; r < reps && (phases & kPhMain); ++r) {
    if (a.ih <= kIT / 2)
      launch_tab_kernel<4, CH>(a, G, s);
    else
      launch_tab_kernel<8, CH>(a, G, s);
    AX_LAUNCHED();
  }
  if (!(phases & kPhFixup) || a.cnt) return hipSuccess;
  // rows of 2^20 blocks: one row of threads of a launch is shorter than 2^32
  const unsigned blocks = (unsigned)ntiles * (unsigned)(a.ih / 64), row = std::min(blocks, 1u << 20);
  const dim3 grid(row, (blocks + row - 1) / row);
  if ((double)a.total_iters * (G + 1) < 4.0e9)  // (w + 1) * total and it * G fit 32 bits
    hipLaunchKernelGGL((tab_fixup_kernel<CH, true>), grid, dim3(256), 0, s, a, G, ntiles);
  else
    hipLaunchKernelGGL((tab_fixup_kernel<CH, false>), grid, dim3(256), 0, s, a, G, ntiles);
  return hipGetLastError();
}

hipError_t launch_tab(const Geom& g, const QParams& qp, const TabPlan& p, const uint8_t* x, const uint8_t* w,
                      const uint16_t* lut, int32_t* acc_out, float* y_out, void* prepared, void* scratch, size_t scratch_bytes,
                      int phases, int main_reps, hipStream_t s) {
  uint8_t* pb = static_cast<uint8_t*>(prepared);
  uint8_t* sb = static_cast<uint8_t*>(scratch);
  const bool ch = (p.variant == 3);
  const int I = ch ? g.Cout : g.M;
  const int J = ch ? g.M : g.Cout;
  const int nchunks = cdiv(g.K, kChunk);
  const int Kp = nchunks * kChunk;
  const int Jpad = cdiv(J, 64) * 64;
  uint16_t* rows = reinterpret_cast<uint16_t*>(pb + p.off_rows);
  QDev* qd = reinterpret_cast<QDev*>(pb + p.off_qd);
  // pixel lanes: packed filters and their sums are constants, the materialized patches per call;
  // channel lanes: the transposed filters are constants, packed patches and their sums per call
  uint8_t* Bp = (ch ? sb : pb) + p.off_bpack;
  int32_t* bsum = reinterpret_cast<int32_t*>((ch ? sb : pb) + p.off_bsum);
  uint8_t* Ap = (ch ? pb : sb) + p.off_apack;

  ConvView cv{x, g.H, g.W, g.Cin, g.KW, g.sh, g.sw, g.ph, g.pw, g.OH, g.OW, g.M, g.K, qp.pad_code, qp.dq,
              g.dh, g.dw, g.sgn ? 0x80u : 0u};

  const int ntiles1 = p.nti * cdiv(J, kJT);  // per table
  const int ntiles = ntiles1 * g.T;
  // Column sums are produced per segment of rows so that more than Jpad/64 blocks share the work.
  const int krows = Kp + 1;
  const int nseg = std::max(1, std::min(kMaxSeg, cdiv(krows, 64)));
  const int seg_rows = cdiv(cdiv(krows, nseg), 16) * 16;
  const int row_blocks = kRowBlocks * g.T, pack_blocks = nseg * (Jpad / 64);
  const bool implicit_view = !ch && reads_in_place(g, x);
  // Activations re-laid out chunk by chunk (prep_chunks_kernel): by output pixel for 1 x 1 filters without
  // padding (only the pixels that are read), else the whole tensor, with its border where the scratch
  // block has room for that (behind the pieces of shared tiles).  Signed codes need a copy in any case, and have
  // the whole block; others are read in place where there is no room.
  const bool by_output = g.KH == 1 && g.KW == 1 && g.ph == 0 && g.pw == 0;
  const double room = scratch_bytes > p.off_apack ? (double)(scratch_bytes - p.off_apack) : 0.0;
  const double bordered = (double)g.N * (g.H + 2.0 * g.ph) * (g.W + 2.0 * g.pw);  // pixels with the border the taps see
  const bool border = !by_output && bordered * g.Cin <= std::min(room, (double)p.ws_apack) && bordered < 268435456.0;  // 16 * pixels: 32 bits
  const bool fits = border || (by_output ? (double)g.M : (double)g.N * g.H * g.W) * g.Cin <= room;
  const bool chunked = implicit_view && (g.sgn || (fits && (g.Cin > 16 || (border && (g.ph || g.pw)))));
  const int bh = chunked && border ? g.ph : 0, bw = chunked && border ? g.pw : 0;
  const int ch_h = by_output ? g.OH : g.H + 2 * bh, ch_w = by_output ? g.OW : g.W + 2 * bw;  // the copy's positions
  uint32_t* rows32 = reinterpret_cast<uint32_t*>(rows);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(pb + p.off_cnt);
  const int ncnt = p.combine ? ntiles : 0;

  if (ch) {
    // one launch when both parts are wanted; otherwise rows + coefficients (+ the transposed
    // filters) as constants, and the packing of the patches per call
    const bool c = phases & kPhConst, k = phases & kPhCall;
    if (c || k) {
      hipLaunchKernelGGL((prep_kernel<true>), dim3((c ? row_blocks : 0) + (k ? pack_blocks : 0)), dim3(256), 0, s, lut,
                         rows32, w, cv, g.K, J, krows, Jpad, seg_rows, Bp, bsum, qp, qd, g.T, c ? 1 : 0, c ? 1 : 0, cnt, ncnt);
      AX_LAUNCHED();
    }
    if (c) {
      hipLaunchKernelGGL(prep_transpose_kernel, dim3(nchunks, cdiv(g.Cout, 1024)), dim3(256), 0, s, w, g.K, g.Cout, Ap, cv.sx);
      AX_LAUNCHED();
    }
  } else {
    if (phases & kPhConst) {
      hipLaunchKernelGGL((prep_kernel<false>), dim3(row_blocks + pack_blocks), dim3(256), 0, s, lut, rows32, w, cv, g.K,
                         J, krows, Jpad, seg_rows, Bp, bsum, qp, qd, g.T, 1, 1, cnt, ncnt);
      AX_LAUNCHED();
    }
    if ((phases & kPhConst) && p.pre) {
      hipLaunchKernelGGL(prep_tables_kernel, dim3((unsigned)(nchunks * (Jpad / 8))), dim3(kThreads), 0, s, rows, Bp, Jpad,
                         pb + p.off_tabs);
      AX_LAUNCHED();
    }
    if ((phases & kPhCall) && chunked) {
      const int pos = g.N * ch_h * ch_w;
      const int cl = g.Cin <= 16 ? 0 : g.Cin <= 32 ? 1 : g.Cin <= 64 ? 2 : 3;
      hipLaunchKernelGGL(prep_chunks_kernel, dim3(cdiv(pos, 512 >> cl), cdiv(g.Cin, 16 << cl)), dim3(256), 0, s, x, pos, g.Cin,
                         cl, g.H, g.W, ch_h * ch_w, ch_w, by_output ? g.sh : 1, by_output ? g.sw : 1, bh, bw,
                         cv.sx * 0x01010101u, qd, Ap);
      AX_LAUNCHED();
    } else if ((phases & kPhCall) && !implicit_view) {
      ConvView rows = cv;
      int images = g.N;
      im2col_flatten(&rows, g.KH, &images);
      Im2colTile t;
      if (im2col_tile(rows, g.KH, images, Kp, &t)) {
        hipLaunchKernelGGL(t.group ? prep_im2col_lds_kernel<true> : prep_im2col_lds_kernel<false>, dim3((unsigned)((long long)images * t.nstripe * t.nrows)), dim3(256),
                           (unsigned)(t.stage_bytes + (size_t)Kp * 2), s, rows, g.KH, nchunks, t, Ap);
      } else {
        const long long pieces = (long long)g.M * (Kp / 16);
        hipLaunchKernelGGL(prep_im2col_kernel, dim3((unsigned)cdiv(pieces, 256)), dim3(256), 0, s, cv, Kp, Ap);
      }
      AX_LAUNCHED();
    }
  }
  const bool fixup = p.partials > 0;
  const int run = (phases & kPhMain) | (fixup ? (phases & kPhFixup) : 0);
  if (!run) return hipSuccess;

  TabArgs a{};
  a.I = I;
  if (implicit_view && !(chunked && by_output)) {
    a.A = chunked ? Ap : x;
    a.H = chunked ? ch_h : g.H; a.W = chunked ? ch_w : g.W; a.Cin = g.Cin; a.KW = g.KW; a.sh = g.sh; a.sw = g.sw;
    a.ph = g.ph - bh; a.pw = g.pw - bw;
    a.OHW = g.OH * g.OW; a.OW = g.OW;
    a.dh = g.dh; a.dw = g.dw;
    a.a_ps = chunked ? 16u : (uint32_t)g.Cin;
    a.a_cs = chunked ? (uint32_t)(g.N * ch_h * ch_w) : 1u;
    // taps outside the image: with padding only (OH and OW count the positions whose taps all lie inside)
    if (a.ph || a.pw) a.padded = g.H + g.ph < 32768 && g.W + g.pw < 32768 ? 1 : 2;
  } else {  // materialized operand: I lane elements of Kp bytes, chunk by chunk, seen as I pixels of a 1 x 1 image
    a.A = Ap;
    a.H = 1; a.W = 1; a.Cin = Kp; a.KW = 1; a.sh = 1; a.sw = 1; a.ph = 0; a.pw = 0; a.OHW = 1; a.OW = 1;
    a.dh = 1; a.dw = 1;
    a.a_ps = 16; a.a_cs = (uint32_t)I;
  }
  a.by_ohw = Divisor(a.OHW); a.by_ow = Divisor(a.OW); a.by_cin = Divisor(a.Cin); a.by_kw = Divisor(a.KW);
  a.Bp = Bp; a.Jpad = Jpad; a.J = J; a.bsum = bsum; a.nseg = cdiv(krows, seg_rows); a.rows = rows;
  a.K = g.K;
  a.ntj = cdiv(J, kJT);
  a.nch = nchunks;
  a.ih = p.ih;
  a.ntiles1 = ntiles1;
  a.total_iters = (long long)ntiles * nchunks;
  a.by_ntiles1 = Divisor(a.ntiles1); a.by_ntj = Divisor(a.ntj); a.by_grid = Divisor(p.G); a.by_nch = Divisor(a.nch);
  a.small = a.total_iters < (1LL << 31) && p.G <= 46340;
  a.share = (int)std::min<long long>(a.total_iters / p.G, 0x7fffffff);
  a.rest = (int)(a.total_iters % p.G);
  a.qd = qd;
  a.bias_k = g.sgn ? 32768u * (uint32_t)g.K : 0u;
  a.acc_out = acc_out; a.y_out = y_out;
  a.part = reinterpret_cast<int32_t*>(sb + p.off_part);
  a.lsum = reinterpret_cast<int32_t*>(sb + p.off_lsum);
  a.cnt = p.combine ? reinterpret_cast<uint32_t*>(pb + p.off_cnt) : nullptr;
  a.tabs = p.pre ? reinterpret_cast<const uint4*>(pb + p.off_tabs) : nullptr;
  a.tabs_bytes = p.pre ? (uint32_t)((size_t)krows * (Jpad / 8) * 4096) : 0u;
  a.out_elems = (long long)g.M * g.Cout;
  a.xcd = p.xcd;
  const uintptr_t outs = (uintptr_t)acc_out | (uintptr_t)y_out;
  a.vec_out = ch ? 0 : J % 4 == 0 && (outs & 15) == 0 ? 2 : J % 2 == 0 && (outs & 7) == 0 ? 1 : 0;

  return ch ? launch_main<true>(a, p.G, ntiles, run, main_reps, s)
            : launch_main<false>(a, p.G, ntiles, run, main_reps, s);
}

}  // namespace ax

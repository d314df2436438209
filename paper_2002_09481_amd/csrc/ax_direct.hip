// Direct kernel: S threads per output element, table read straight from global memory.
//
// This is the simplest device formulation of the layer (Sec. II Eq. (3)/(4) with the product
// replaced by the truth-table entry; Sec. III layouts): consecutive lanes take consecutive
// output channels of one pixel, so the activation code is wave-uniform, the filter codes
// are a coalesced 64-byte read and the lookups fall into one 512-byte table row.  It is
// used for tiny problems and for shapes the table-tile kernels do not take.
#include <algorithm>
#include <cmath>

#include "ax_internal.h"

namespace ax {

// Tiny problems give few threads, each with a serial chain of dependent loads (code, then entry), so
// their time is that chain and not any bandwidth: S threads of a block share the taps of an output
// (thread s takes the taps s, s + S, ...) and their sums meet in LDS.  S = 1 against S by
// direct_threads, calls in a chain on the device: 16 x 16 x 8 3 x 3 to 8 channels 17.3 -> 5.0 us, dense
// 500 x 100 x 30 21.7 -> 7.8 us.
template <int S>
__global__ __launch_bounds__(256) void direct_kernel(Geom g, QParams qp_in, const uint8_t* __restrict__ x,
                                                      const uint8_t* __restrict__ w,
                                                      const uint16_t* __restrict__ lut,
                                                      int32_t* __restrict__ acc_out,
                                                      float* __restrict__ y_out) {
  QParams qp = qp_in;
  if (qp.dq) {  // coefficients produced on the device
    qp.x_zp = qp.dq->x_zp;
    qp.w_zp = qp.dq->w_zp;
    qp.pad_code = qp.x_zp;
    qp.scale = qp.dq->x_scale * qp.dq->w_scale;
  }
  const uint32_t total = (uint32_t)g.M * (uint32_t)g.Cout;
  constexpr uint32_t OUT = 256u / S;  // outputs per block
  const uint32_t oi = threadIdx.x % OUT, slice = threadIdx.x / OUT;
  const uint32_t o = blockIdx.x * OUT + oi;
  if (S == 1 && o >= total) return;
  const uint32_t oc = min(o, total - 1u);
  const int co = oc % (uint32_t)g.Cout;
  uint32_t m = oc / (uint32_t)g.Cout;
  const int ox = m % (uint32_t)g.OW;
  m /= (uint32_t)g.OW;
  const int oy = m % (uint32_t)g.OH;
  const int n = m / (uint32_t)g.OH;

  // Channel blocks: output channel co of block co / (Cout / groups) sums over the taps of that
  // block's Cin / groups input channels; filters are [KH, KW, Cin / groups, Cout].  One block is
  // the ordinary layer; the depthwise layer is the case of one input channel per block (its
  // filters [KH, KW, Cin, mult] are the same bytes).
  const int c_count = g.Cin / g.groups;
  const int c_first = (co / (g.Cout / g.groups)) * c_count;
  const int wcols = g.Cout;  // innermost extent of the filter tensor
  const int wcol = co;
  // Signed codes are sign-extended bytes; the table is addressed by their 8-bit patterns and
  // its entries are sign-extended too.
  int32_t acc = 0, sp = 0, sf = 0;
  auto add = [&](uint32_t ap, uint32_t bp) {
    const uint32_t e = lut[ap * 256u + bp];
    if (g.sgn) {
      acc += (int32_t)(int16_t)e;
      sp += (int32_t)(int8_t)ap;
      sf += (int32_t)(int8_t)bp;
    } else {
      acc += (int32_t)e;  // sums stay below 2^31 (K <= 32768)
      sp += (int32_t)ap;
      sf += (int32_t)bp;
    }
  };
  if constexpr (S == 1) {
    for (int ky = 0; ky < g.KH; ++ky) {
      const int iy = oy * g.sh - g.ph + ky * g.dh;
      for (int kx = 0; kx < g.KW; ++kx) {
        const int ix = ox * g.sw - g.pw + kx * g.dw;
        const bool inside = (iy >= 0) && (iy < g.H) && (ix >= 0) && (ix < g.W);
        const uint8_t* xp = x + (((size_t)n * g.H + (inside ? iy : 0)) * g.W + (inside ? ix : 0)) * g.Cin + c_first;
        const uint8_t* wp = w + (size_t)(ky * g.KW + kx) * c_count * wcols + wcol;
        for (int ci = 0; ci < c_count; ++ci)
          add(inside ? (uint32_t)xp[ci] : ((uint32_t)qp.pad_code & 0xffu), wp[(size_t)ci * wcols]);
      }
    }
  } else {
    // batches of eight taps: all their codes are requested before the first entry is looked up
    constexpr int B = 8;
    for (int k0 = (int)slice; k0 < g.K; k0 += B * S) {
      uint32_t ap[B], bp[B];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const uint32_t k = (uint32_t)min(k0 + b * S, g.K - 1);
        const uint32_t tap = k / (uint32_t)c_count, ci = k - tap * (uint32_t)c_count;
        const uint32_t ky = tap / (uint32_t)g.KW, kx = tap - ky * (uint32_t)g.KW;
        const int iy = oy * g.sh - g.ph + (int)ky * g.dh, ix = ox * g.sw - g.pw + (int)kx * g.dw;
        const bool inside = (iy >= 0) && (iy < g.H) && (ix >= 0) && (ix < g.W);
        const uint32_t v = x[(((size_t)n * g.H + (inside ? iy : 0)) * g.W + (inside ? ix : 0)) * g.Cin + c_first + ci];
        ap[b] = inside ? v : ((uint32_t)qp.pad_code & 0xffu);
        bp[b] = w[(size_t)k * wcols + wcol];
      }
#pragma unroll
      for (int b = 0; b < B; ++b)
        if (k0 + b * S < g.K) add(ap[b], bp[b]);
    }
    __shared__ int32_t part[3][256];
    part[0][threadIdx.x] = acc;
    part[1][threadIdx.x] = sp;
    part[2][threadIdx.x] = sf;
    __syncthreads();
    if (slice != 0 || o >= total) return;
#pragma unroll 8
    for (uint32_t i = 1; i < (uint32_t)S; ++i) {
      acc += part[0][oi + i * OUT];
      sp += part[1][oi + i * OUT];
      sf += part[2][oi + i * OUT];
    }
  }
  if (acc_out) acc_out[o] = acc;
  if (y_out) {
    const long long corr = (long long)acc - (long long)qp.w_zp * sp - (long long)qp.x_zp * sf +
                           (long long)g.K * qp.x_zp * qp.w_zp;
    y_out[o] = (float)corr * qp.scale;
  }
}

// Depthwise layers.  No table-side operand is shared between output channels, so the table-tile
// scheme does not apply; instead every workgroup keeps the whole 128 KB table in LDS (one
// workgroup of 1024 threads per compute unit) and gathers 2-byte entries at data-dependent
// addresses.  One thread takes 4 consecutive output channels of one output pixel and stores 16
// bytes per output tensor.  Signed tables are stored with 32768 added to every entry and activation
// sums are taken over the byte patterns with the top bit flipped (code + 128); both offsets come
// off again in the epilogue.
//
// Table rows (one per activation code) are kDwRow = 129 dwords apart, not 128: with a stride of
// 128 dwords the LDS bank of an entry depends on the filter code alone, and the lanes of a wave
// that work on the same channels of different pixels (same filter codes, different activation
// codes) would all fall into one bank.  With the odd stride the bank is (activation code +
// filter code / 2) mod 64, as good as random.
constexpr int kDwMaxC = 4096;  // output channels whose filter sums fit next to the table in LDS
constexpr int kDwRow = 129;    // dwords per table row in LDS

// KS: kernel height = width known at compile time (taps fully unrolled, so that the loads of all
// taps of an item are in flight together), or 0 for any kernel size.
// GEN: any channel multiplier and channel count: output channel co reads input channel co / mult and
// filter code w[tap * Cout + co]; codes are loaded byte by byte and the last group of a pixel may
// hold fewer than four channels.  Otherwise multiplier 1 and Cin % 4 == 0: one dword per tap and operand.
template <int KS, bool GEN>
__global__ __launch_bounds__(1024) void dw_kernel(Geom g, QParams qp_in, const uint8_t* __restrict__ x,
                                                   const uint8_t* __restrict__ w, const uint16_t* __restrict__ lut,
                                                   int32_t* __restrict__ acc_out, float* __restrict__ y_out,
                                                   int vec_out) {
  __shared__ uint32_t tab[256 * kDwRow];
  __shared__ int32_t sfs[kDwMaxC];  // per output channel: sum over the taps of the filter codes (+128 each if signed)
  QParams qp = qp_in;
  if (qp.dq) {
    qp.x_zp = qp.dq->x_zp;
    qp.w_zp = qp.dq->w_zp;
    qp.pad_code = qp.x_zp;
    qp.scale = qp.dq->x_scale * qp.dq->w_scale;
  }
  const uint32_t flip16 = g.sgn ? 0x80008000u : 0u;
  const uint32_t flip8 = g.sgn ? 0x80808080u : 0u;
  const int KH = KS ? KS : g.KH, KW = KS ? KS : g.KW;
  const int K = KH * KW;
  {
    const uint4* __restrict__ src = reinterpret_cast<const uint4*>(lut);
    // signed activations index the table by code + 128 (the byte with its top bit flipped), the
    // same value the patch sums are taken over: rows are staged in that order (a row = 32 chunks)
    const int rowflip = g.sgn ? (0x80 << 5) : 0;
    for (int i = threadIdx.x; i < 8192; i += 1024) {
      uint4 v = src[i ^ rowflip];
      uint32_t* dst = tab + (i >> 5) * kDwRow + (i & 31) * 4;
      dst[0] = v.x ^ flip16; dst[1] = v.y ^ flip16; dst[2] = v.z ^ flip16; dst[3] = v.w ^ flip16;
    }
    for (int c = threadIdx.x; c < g.Cout; c += 1024) {
      int32_t t = 0;
      for (int k = 0; k < K; ++k) t += (int32_t)((uint32_t)w[(size_t)k * g.Cout + c] ^ (flip8 & 0xffu));
      sfs[c] = t;
    }
  }
  __syncthreads();
  const uint32_t C4 = ((uint32_t)g.Cout + 3u) / 4u;  // groups of four output channels per pixel
  const uint32_t items = (uint32_t)g.M * C4;          // M * Cout < 2^31
  const uint32_t padb = ((uint32_t)qp.pad_code & 0xffu);
  const uint32_t pad4 = padb * 0x01010101u;
  const uint32_t bias = g.sgn ? 32768u * (uint32_t)K : 0u;
  const int off128 = g.sgn ? 128 * K : 0;
  const long long kzz = (long long)K * qp.x_zp * qp.w_zp;
  const char* tabb = reinterpret_cast<const char*>(tab);
  auto entry = [&](uint32_t a, uint32_t b2) -> uint32_t {  // b2 = 2 * filter code
    return *reinterpret_cast<const uint16_t*>(tabb + (a * (uint32_t)(kDwRow * 4) + b2));
  };
  for (uint32_t it = blockIdx.x * 1024u + threadIdx.x; it < items; it += gridDim.x * 1024u) {
    const uint32_t c4 = it % C4;
    const uint32_t pix = it / C4;
    uint32_t m = pix;
    const int ox = m % (uint32_t)g.OW;
    m /= (uint32_t)g.OW;
    const int oy = m % (uint32_t)g.OH;
    const int n = m / (uint32_t)g.OH;
    const int by = oy * g.sh - g.ph, bx = ox * g.sw - g.pw;
    uint32_t acc[4] = {0, 0, 0, 0};
    uint32_t sp[4] = {0, 0, 0, 0};
    auto tap = [&](uint32_t xd, uint32_t wd) {
      const uint32_t xs = xd ^ flip8;  // code + 128 for signed codes
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t a = (xs >> (8 * j)) & 0xffu, b = (wd >> (8 * j)) & 0xffu;
        acc[j] += entry(a, b << 1);
        sp[j] += a;
      }
    };
    if constexpr (GEN) {
      // output channels co0 .. co0 + 3 (clamped for the last group), their input channels and the
      // position of their filter codes within a tap
      uint32_t co[4], ci[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        co[j] = min(4u * c4 + (uint32_t)j, (uint32_t)g.Cout - 1u);
        ci[j] = co[j] / (uint32_t)g.mult;
      }
      const uint8_t* __restrict__ xn = x + (size_t)n * g.H * g.W * g.Cin;
      for (int ky = 0; ky < KH; ++ky) {
        const int iy = by + ky * g.dh;
        for (int kx = 0; kx < KW; ++kx) {
          const int ix = bx + kx * g.dw;
          const bool inside = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
          const uint8_t* xp = xn + ((size_t)(inside ? iy : 0) * g.W + (inside ? ix : 0)) * g.Cin;
          const uint8_t* wp = w + (size_t)(ky * KW + kx) * g.Cout;
          uint32_t xd = 0, wd = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            xd |= (inside ? (uint32_t)xp[ci[j]] : padb) << (8 * j);
            wd |= (uint32_t)wp[co[j]] << (8 * j);
          }
          tap(xd, wd);
        }
      }
    } else {
      const uint8_t* __restrict__ xn = x + (size_t)n * g.H * g.W * g.Cin + 4u * c4;
      const uint8_t* __restrict__ wc = w + 4u * c4;
      if constexpr (KS > 0) {
        uint32_t xd[KS * KS], wd[KS * KS];
#pragma unroll
        for (int ky = 0; ky < KS; ++ky) {
#pragma unroll
          for (int kx = 0; kx < KS; ++kx) {
            const int iy = by + ky * g.dh, ix = bx + kx * g.dw;
            const bool inside = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
            xd[ky * KS + kx] = pad4;
            if (inside) xd[ky * KS + kx] = *reinterpret_cast<const uint32_t*>(xn + ((size_t)iy * g.W + ix) * g.Cin);
            wd[ky * KS + kx] = *reinterpret_cast<const uint32_t*>(wc + (size_t)(ky * KS + kx) * g.Cin);
          }
        }
#pragma unroll
        for (int t = 0; t < KS * KS; ++t) tap(xd[t], wd[t]);
      } else {
        for (int ky = 0; ky < KH; ++ky) {
          const int iy = by + ky * g.dh;
          for (int kx = 0; kx < KW; ++kx) {
            const int ix = bx + kx * g.dw;
            const bool inside = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
            uint32_t xd = pad4;
            if (inside) xd = *reinterpret_cast<const uint32_t*>(xn + ((size_t)iy * g.W + ix) * g.Cin);
            tap(xd, *reinterpret_cast<const uint32_t*>(wc + (size_t)(ky * KW + kx) * g.Cin));
          }
        }
      }
    }
    int32_t av[4];
    float yv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int32_t sf = sfs[min(4u * c4 + (uint32_t)j, (uint32_t)g.Cout - 1u)];
      av[j] = (int32_t)(acc[j] - bias);
      if (g.K <= 4096) {  // every term below 2^29: 32-bit arithmetic is exact
        const int32_t corr = av[j] - (int32_t)qp.w_zp * ((int32_t)sp[j] - off128) - (int32_t)qp.x_zp * (sf - off128) + (int32_t)kzz;
        yv[j] = (float)corr * qp.scale;
      } else {
        const long long corr = (long long)av[j] - (long long)qp.w_zp * ((int32_t)sp[j] - off128) -
                               (long long)qp.x_zp * (sf - off128) + kzz;
        yv[j] = (float)corr * qp.scale;
      }
    }
    const size_t o = (size_t)pix * g.Cout + 4u * c4;
    if (vec_out) {  // Cout % 4 == 0 and 16-byte aligned outputs
      if (acc_out) *reinterpret_cast<int4*>(acc_out + o) = make_int4(av[0], av[1], av[2], av[3]);
      if (y_out) *reinterpret_cast<float4*>(y_out + o) = make_float4(yv[0], yv[1], yv[2], yv[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (4u * c4 + (uint32_t)j < (uint32_t)g.Cout) {
          if (acc_out) acc_out[o + j] = av[j];
          if (y_out) y_out[o + j] = yv[j];
        }
      }
    }
  }
}

// 3 x 3 depthwise layers with multiplier 1 and a channel count divisible by four: every thread keeps
// its four channels, so the filter codes stay pre-shifted in registers; PX items (pixels) per thread
// and iteration.  All loads of the PX items are issued before the first lookup, so that a wave has PX
// times the lookups to cover one memory round trip with (the workgroup fills the compute unit's LDS, so
// more waves are not to be had).
// Bound: vector issue, about as much for the addresses of the codes as for the lookups, and the gathers:
// the vector units issue in 73 % of the busy cycles, the LDS is active in 72 %.  So the position of an item is carried on by additions (no divisions) and a tap
// is one 32-bit offset from a uniform step; a lookup is a byte extract and one multiply-add, which
// took half-rate sub-dword multiplies before.  The first codes and the filters travel while the
// table is staged.  112 x 112 x 32 at batch 32: 37.1 -> 32.4 us, both outputs written.
// Channel-group counts that do not divide 1024, on the general kernel before -> here, batch 32:
// 56 x 56 x 96 37.6 -> 26.9 us, 14 x 14 x 576 19.5 -> 15.6 us, 56 x 56 x 144 stride 2 19.4 -> 16.1 us.
template <int PX>
__global__ __launch_bounds__(1024) void dw3_kernel(Geom g, QParams qp_in, const uint8_t* __restrict__ x,
                                                    const uint8_t* __restrict__ w, const uint16_t* __restrict__ lut,
                                                    int32_t* __restrict__ acc_out, float* __restrict__ y_out,
                                                    int vec_out) {
  __shared__ uint32_t tab[256 * kDwRow];
  __shared__ int32_t sfs[kDwMaxC];
  QParams qp = qp_in;
  if (qp.dq) {
    qp.x_zp = qp.dq->x_zp;
    qp.w_zp = qp.dq->w_zp;
    qp.pad_code = qp.x_zp;
    qp.scale = qp.dq->x_scale * qp.dq->w_scale;
  }
  const uint32_t flip16 = g.sgn ? 0x80008000u : 0u;
  const uint32_t flip8 = g.sgn ? 0x80808080u : 0u;
  const uint32_t C4 = (uint32_t)g.Cout / 4u;
  const uint32_t items = (uint32_t)g.M * C4;
  const uint32_t pad4 = ((uint32_t)qp.pad_code & 0xffu) * 0x01010101u;
  // the grid stride is a multiple of the channel groups; the up to C4 - 1 threads beyond it get no item
  const uint32_t stride = gridDim.x * 1024u / C4 * C4;
  const uint32_t tid = blockIdx.x * 1024u + threadIdx.x;
  const uint32_t gid = tid < stride ? tid : items + tid;
  const uint32_t c4 = gid % C4;  // the same for every item of this thread: stride % C4 == 0
  // Position of the next item to load and the way from one item to the next (the same for all threads).
  uint32_t nx = gid;  // its number
  int ox, oy, n;
  const uint32_t step = stride / C4;  // pixels
  const int step_x = step % (uint32_t)g.OW, step_r = step / (uint32_t)g.OW;
  const int step_y = step_r % g.OH, step_n = step_r / g.OH;
  {
    uint32_t m = gid / C4;
    ox = m % (uint32_t)g.OW;
    m /= (uint32_t)g.OW;
    oy = m % (uint32_t)g.OH;
    n = m / (uint32_t)g.OH;
  }
  const uint32_t dx = (uint32_t)g.dw * (uint32_t)g.Cin, dy = (uint32_t)g.dh * (uint32_t)g.W * (uint32_t)g.Cin;
  uint32_t xd[PX][9];
  auto load = [&]() {  // the next PX items; offsets into x are below 2^31
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const int by = oy * g.sh - g.ph, bx = ox * g.sw - g.pw;
      const uint32_t base = (uint32_t)((n * g.H + by) * g.W + bx) * (uint32_t)g.Cin + 4u * c4;
      const bool valid = nx < items;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) {
        const bool in_y = valid && (unsigned)(by + ky * g.dh) < (unsigned)g.H;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
          const bool inside = in_y && (unsigned)(bx + kx * g.dw) < (unsigned)g.W;
          const uint32_t v = *reinterpret_cast<const uint32_t*>(x + (inside ? base + (ky * dy + kx * dx) : 0u));
          xd[p][ky * 3 + kx] = inside ? v : pad4;
        }
      }
      nx += stride;
      ox += step_x;
      const bool cx = ox >= g.OW;
      ox -= cx ? g.OW : 0;
      oy += step_y + (cx ? 1 : 0);
      const bool cy = oy >= g.OH;
      oy -= cy ? g.OH : 0;
      n += step_n + (cy ? 1 : 0);
    }
  };
  // the first codes travel while the table is staged
  load();
  uint32_t wb2[9][4];  // 2 * filter code = byte offset within a table row
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const uint32_t wd = *reinterpret_cast<const uint32_t*>(w + (size_t)t * g.Cin + 4u * c4);
#pragma unroll
    for (int j = 0; j < 4; ++j) wb2[t][j] = ((wd >> (8 * j)) & 0xffu) << 1;
  }
  {
    const uint4* __restrict__ src = reinterpret_cast<const uint4*>(lut);
    const int rowflip = g.sgn ? (0x80 << 5) : 0;  // see dw_kernel
#pragma unroll 4
    for (int i0 = 0; i0 < 8192; i0 += 1024) {
      const int i = i0 + threadIdx.x;
      const uint4 v = src[i ^ rowflip];
      uint32_t* dst = tab + (i >> 5) * kDwRow + (i & 31) * 4;
      dst[0] = v.x ^ flip16; dst[1] = v.y ^ flip16; dst[2] = v.z ^ flip16; dst[3] = v.w ^ flip16;
    }
    for (int c = threadIdx.x; c < g.Cout; c += 1024) {
      int32_t t = 0;
      for (int k = 0; k < 9; ++k) t += (int32_t)((uint32_t)w[(size_t)k * g.Cout + c] ^ (flip8 & 0xffu));
      sfs[c] = t;
    }
  }
  __syncthreads();
  const uint32_t bias = g.sgn ? 32768u * 9u : 0u;
  const int off128 = g.sgn ? 128 * 9 : 0;
  const long long kzz = 9LL * qp.x_zp * qp.w_zp;
  const char* tabb = reinterpret_cast<const char*>(tab);
  int32_t xz_sf[4];  // x_zp * (sum of the channel's filter codes): constant per thread
#pragma unroll
  for (int j = 0; j < 4; ++j) xz_sf[j] = (int32_t)qp.x_zp * (sfs[4u * c4 + j] - off128);
  const int32_t kzz32 = (int32_t)kzz;
  const uint32_t rowbytes = (uint32_t)(kDwRow * 4);
  for (uint32_t it0 = gid; it0 < items;) {
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const uint32_t it = it0 + p * stride;
      if (it >= items) break;
      // Per lookup: extract the code, offset = code * 516 + column offset in one multiply-add, gather;
      // the sums of the entries and of the codes take two taps per instruction.
      uint32_t acc[4] = {0, 0, 0, 0}, sp[4] = {0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const uint32_t xs = xd[p][t] ^ flip8;  // code + 128 for signed codes
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t a = (xs >> (8 * j)) & 0xffu;
          acc[j] += *reinterpret_cast<const uint16_t*>(tabb + (__umul24(a, rowbytes) + wb2[t][j]));
          sp[j] += a;
        }
      }
      int32_t av[4];
      float yv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        av[j] = (int32_t)(acc[j] - bias);
        // nine taps: every term is below 2^20, 32-bit arithmetic is exact
        const int32_t corr = av[j] - (int32_t)qp.w_zp * ((int32_t)sp[j] - off128) - xz_sf[j] + kzz32;
        yv[j] = (float)corr * qp.scale;
      }
      const size_t o = (size_t)it * 4u;  // = pixel * Cout + 4 * c4
      if (vec_out) {  // 16-byte aligned outputs
        if (acc_out) *reinterpret_cast<int4*>(acc_out + o) = make_int4(av[0], av[1], av[2], av[3]);
        if (y_out) *reinterpret_cast<float4*>(y_out + o) = make_float4(yv[0], yv[1], yv[2], yv[3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (acc_out) acc_out[o + j] = av[j];
          if (y_out) y_out[o + j] = yv[j];
        }
      }
    }
    it0 += PX * stride;
    if (it0 < items) load();
  }
}

// Layers of few output pixels (the deep layers of a network at batch 1, a fully connected layer at a
// small batch).  A table tile would spend more on assembling its tables than on the lookups they
// serve; here every workgroup keeps the whole table in LDS, as the depthwise kernel does, and
// gathers 2-byte entries.  A tile is P pixels x 4 CL output channels, the taps are cut into 1024 / CL
// slices of four consecutive taps in turn: a lane reads one dword of activations per pixel and one
// dword of filter codes per tap and makes 16 P lookups of them, so that a lookup costs one address
// addition, one gather and one accumulation.  Lanes of neighbouring slices lie side by side; their
// sums meet in DPP additions, those of the waves in 64-bit LDS atomics (two 32-bit sums at a time,
// neither reaches 2^32; integer, any order gives the same bits).  One launch, no preparation, no
// scratch.  Workgroups walk over tiles, so a table is staged once per compute unit.
// Bound: waits.  On the layers of the ResNet-50 shape at batch 1 the LDS is active in 63 % of the
// cycles of the busy compute units (38 % bank conflicts of the random 2-byte gathers), the vector units
// issue in 54 %, and a wave waits in 57 % of its cycles: for its own gathers, of which at most two are in
// flight, and at the barriers between staging, lookups, sums and stores.  3.3 to 4.2 T lookups/s after
// about 5 us of launch and staging; the gathers alone would allow 5.2 T/s.
// Measured, calls in a chain on the device, before (T: table tiles, D: direct_kernel with one thread per
// output, F: a kernel for dense layers of few rows) -> here: 7 x 7 x 512 3 x 3 T 111.5 -> 32.8 us,
// 14 x 14 x 256 3 x 3 T 42.4 -> 32.2 us, 14 x 14 x 1024 1 x 1 to 256 T 28.5 -> 20.8 us, dense
// 1 x 2048 x 1000 D 378 -> 7.6 us, 8 x 4096 x 4096 F 173 -> 40.6 us, 32 x 2048 x 1000 F 26.9 -> 23.6 us.
// Eight pixels of four channels (32 sums) are what 128 registers hold with a step's codes in flight.
// DWORDS: Cin % 4 == 0: four consecutive taps are one dword of one pixel.
// Operands may start at any byte and tables at any entry, and Cout need not be a multiple of four: dwords
// and the staged pieces of the table are loaded at their own alignment (load_any), the last dword of a
// filter row ends with the row.  Byte by byte instead, x off a dword boundary took 63 us against 40.5 us
// on the table tiles (396 x 128 x 2001; 32.8 us now, 33 us aligned), filter rows of 1001 codes 49.2 us
// against 32.2 us (8 x 8192).
template <int P, bool DWORDS>
__global__ __launch_bounds__(1024) void fewpix_kernel(Geom g, QParams qp_in, const uint8_t* __restrict__ x,
                                                       const uint8_t* __restrict__ w, const uint16_t* __restrict__ lut,
                                                       int32_t* __restrict__ acc_out, float* __restrict__ y_out,
                                                       int cl_log2) {
  __shared__ uint32_t tab[256 * kDwRow];
  __shared__ __align__(16) uint32_t accs[P * 256];  // [pixel][channel of the tile]
  __shared__ uint32_t sps[P], sfs[256];
  QParams qp = qp_in;
  if (qp.dq) {
    qp.x_zp = qp.dq->x_zp;
    qp.w_zp = qp.dq->w_zp;
    qp.pad_code = qp.x_zp;
    qp.scale = qp.dq->x_scale * qp.dq->w_scale;
  }
  const uint32_t flip8 = g.sgn ? 0x80808080u : 0u;
  const uint32_t pad4 = ((uint32_t)qp.pad_code & 0xffu) * 0x01010101u;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sl_log2 = 6 - cl_log2;                  // slices side by side in a wave
  const int cl = lane >> sl_log2;                   // channel group of the lane
  const int CT = 4 << cl_log2;                      // channels per tile
  const int slices = 1024 >> cl_log2;
  const int slice = (wave << sl_log2) + (lane & ((1 << sl_log2) - 1));
  const int K = g.K, J = g.Cout, M = g.M;
  const int K4 = (K + 3) >> 2;
  const int nct = (J + CT - 1) / CT, ntiles = nct * ((M + P - 1) / P);
  for (int i = threadIdx.x; i < P * 256; i += 1024) accs[i] = 0;
  if (threadIdx.x < 256) sfs[threadIdx.x] = 0;
  if (threadIdx.x < P) sps[threadIdx.x] = 0;
  const char* tabb = reinterpret_cast<const char*>(tab);
  const uint32_t rowbytes = (uint32_t)(kDwRow * 4);

  int j0, m0, wcol, by[P], bx[P], nb[P];
  uint32_t wshift;
  // Channel tiles go fastest: workgroup b runs on XCD b mod 8, so where their number is a multiple of
  // eight each XCD's L2 fetches one eighth of the filters.
  auto locate = [&](int tile) {
    const int pt = tile / nct;
    j0 = (tile - pt * nct) * CT;
    m0 = pt * P;
    // the lane's four channels; where fewer are left the dword ends with the filter row and its surplus
    // is shifted out (lanes wholly beyond the row get some codes, whose sums are not stored)
    const int co0 = j0 + 4 * cl;
    wcol = min(co0, J - 4);
    wshift = (8u * (uint32_t)(co0 - wcol)) & 31u;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int m = min(m0 + p, M - 1);
      const int n = m / (g.OH * g.OW), r = m - n * (g.OH * g.OW);
      const int oy = r / g.OW;
      by[p] = oy * g.sh - g.ph;
      bx[p] = (r - oy * g.OW) * g.sw - g.pw;
      nb[p] = n * g.H;
    }
  };
  // offsets into x and w are below 2^31
  auto load = [&](int k4, uint32_t (&xd)[P], uint32_t (&wd)[4]) {
    const int k = 4 * k4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      wd[e] = load_any<uint32_t>(w + ((uint32_t)min(k + e, K - 1) * (uint32_t)J + (uint32_t)wcol)) >> (DWORDS ? 0 : wshift);
    if constexpr (DWORDS) {
      const int tap = k / g.Cin, ci = k - tap * g.Cin;
      const int ky = tap / g.KW, kx = tap - ky * g.KW;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int iy = by[p] + ky * g.dh, ix = bx[p] + kx * g.dw;
        const bool inside = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
        const uint32_t pix = inside ? (uint32_t)(nb[p] + iy) * (uint32_t)g.W + (uint32_t)ix : 0u;
        const uint32_t v = load_any<uint32_t>(x + (pix * (uint32_t)g.Cin + (uint32_t)ci));
        xd[p] = inside ? v : pad4;
      }
    } else {
#pragma unroll
      for (int p = 0; p < P; ++p) xd[p] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ke = min(k + e, K - 1);
        const int tap = ke / g.Cin, ci = ke - tap * g.Cin;
        const int ky = tap / g.KW, kx = tap - ky * g.KW;
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const int iy = by[p] + ky * g.dh, ix = bx[p] + kx * g.dw;
          const bool inside = (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
          const uint32_t pix = inside ? (uint32_t)(nb[p] + iy) * (uint32_t)g.W + (uint32_t)ix : 0u;
          const uint32_t v = x[pix * (uint32_t)g.Cin + (uint32_t)ci];
          xd[p] |= (inside ? v : (pad4 & 0xffu)) << (8 * e);
        }
      }
    }
  };
  uint32_t xd[P], wd[4];
  int tile = blockIdx.x;  // the grid has no more workgroups than there are tiles
  // the first codes travel while the table is staged (the byte form, which assembles its dwords at once,
  // would wait for them)
  if constexpr (DWORDS) {
    locate(tile);
    if (slice < K4) load(slice, xd, wd);
  }
  {
    // signed activations index the table by code + 128: rows are staged in that order, entries with
    // 32768 added (both come off again in the epilogue), as in dw_kernel
    const uint32_t flip16 = g.sgn ? 0x80008000u : 0u;
    const int rowflip = g.sgn ? (0x80 << 5) : 0;
    uint4 piece[8];  // all in flight together
#pragma unroll
    for (int n = 0; n < 8; ++n) piece[n] = load_any<uint4>(lut + 8 * ((n * 1024 + (int)threadIdx.x) ^ rowflip));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int i = n * 1024 + threadIdx.x;
      const uint4 v = piece[n];
      uint32_t* dst = tab + (i >> 5) * kDwRow + (i & 31) * 4;
      dst[0] = v.x ^ flip16; dst[1] = v.y ^ flip16; dst[2] = v.z ^ flip16; dst[3] = v.w ^ flip16;
    }
    __syncthreads();
  }
  for (;;) {
    if constexpr (!DWORDS) {
      locate(tile);
      if (slice < K4) load(slice, xd, wd);
    }
    uint32_t acc[P][4], sp[P], sf[4] = {0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < P; ++p) {
      sp[p] = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[p][j] = 0;
    }
    for (int k4 = slice; k4 < K4; k4 += slices) {
      uint32_t xs[P], ws[4];
#pragma unroll
      for (int p = 0; p < P; ++p) xs[p] = xd[p] ^ flip8;
#pragma unroll
      for (int e = 0; e < 4; ++e) ws[e] = wd[e] >> (DWORDS ? wshift : 0);  // the byte form waits for its codes anyway
      if (k4 + slices < K4) load(k4 + slices, xd, wd);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!DWORDS && 4 * k4 + e >= K) break;
        uint32_t wb2[4];  // 2 * filter code = byte offset within a table row
#pragma unroll
        for (int j = 0; j < 4; ++j) wb2[j] = (j ? ws[e] >> (8 * j - 1) : ws[e] << 1) & 0x1feu;
        const uint32_t wf = ws[e] ^ flip8;  // code + 128 for signed codes
#pragma unroll
        for (int j = 0; j < 4; ++j) sf[j] += (wf >> (8 * j)) & 0xffu;
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const uint32_t a = (xs[p] >> (8 * e)) & 0xffu;
          sp[p] += a;
          const uint32_t row = __umul24(a, rowbytes);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            // an instruction, since the optimizer turns the sums over an unrolled step into trees that
            // keep every gathered entry alive
            const uint32_t v = *reinterpret_cast<const uint16_t*>(tabb + (row + wb2[j]));
            asm("v_add_u32 %0, %1, %0" : "+v"(acc[p][j]) : "v"(v));
          }
        }
        // one tap's gathers in flight at a time: more of them would not fit the registers
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the next tile's first codes travel while this one's sums meet (3 % of a call of several rounds)
    const int mt = m0, jt = j0;
    tile += (int)gridDim.x;
    const bool more = tile < ntiles;  // uniform
    if (DWORDS && more) {
      locate(tile);
      if (slice < K4) load(slice, xd, wd);
    }
    // Sums over the slices that lie side by side in the wave, within rows of 16 lanes: afterwards every
    // lane of a group of 1 << dpp_log2 holds them.  After the first steps the lanes of a quad (of
    // eight) are equal, so the mirrored lane stands for the lane of the other half.
    const int dpp_log2 = min(sl_log2, 4);
    auto wave_sum = [&](uint32_t v) -> uint32_t {
      if (dpp_log2 > 0) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);   // lane ^ 1
      if (dpp_log2 > 1) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);   // lane ^ 2
      if (dpp_log2 > 2) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true);  // mirrored in 8
      if (dpp_log2 > 3) v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, true);  // mirrored in 16
      return v;
    };
#pragma unroll
    for (int p = 0; p < P; ++p) {
      sp[p] = wave_sum(sp[p]);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[p][j] = wave_sum(acc[p][j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) sf[j] = wave_sum(sf[j]);
    if ((lane & ((1 << dpp_log2) - 1)) == 0) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        unsigned long long* dst = reinterpret_cast<unsigned long long*>(accs + p * 256 + 4 * cl);
        atomicAdd(dst, acc[p][0] | ((unsigned long long)acc[p][1] << 32));
        atomicAdd(dst + 1, acc[p][2] | ((unsigned long long)acc[p][3] << 32));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) atomicAdd(&sfs[4 * cl + j], sf[j]);
      if (cl == 0) {
#pragma unroll
        for (int p = 0; p < P; ++p) atomicAdd(&sps[p], sp[p]);
      }
    }
    __syncthreads();
    const uint32_t bias = g.sgn ? 32768u * (uint32_t)K : 0u;
    const int off128 = g.sgn ? 128 * K : 0;
    const long long kzz = (long long)K * qp.x_zp * qp.w_zp;
    for (int i = threadIdx.x; i < P * CT; i += 1024) {
      const int p = i >> (cl_log2 + 2), c = i & (CT - 1);
      if (mt + p < M && jt + c < J) {
        const int32_t av = (int32_t)(accs[p * 256 + c] - bias);
        const size_t o = (size_t)(mt + p) * J + jt + c;
        if (acc_out) acc_out[o] = av;
        if (y_out) {
          const long long corr = (long long)av - (long long)qp.w_zp * ((int32_t)sps[p] - off128) -
                                 (long long)qp.x_zp * ((int32_t)sfs[c] - off128) + kzz;
          y_out[o] = (float)corr * qp.scale;
        }
      }
    }
    if (!more) break;
    __syncthreads();
    for (int i = threadIdx.x; i < P * CT; i += 1024) accs[(i >> (cl_log2 + 2)) * 256 + (i & (CT - 1))] = 0;
    if (threadIdx.x < 256) sfs[threadIdx.x] = 0;
    if (threadIdx.x < P) sps[threadIdx.x] = 0;
    __syncthreads();
  }
}

FewpixPlan fewpix_plan(const Geom& g) {
  const bool dwords = g.Cin % 4 == 0;
  static const int kPixels[] = {1, 2, 4, 7, 8};  // 7: images of 7 x 7, 14 x 14, 28 x 28 ... pixels
  const int K4 = (g.K + 3) / 4, cus = cu_count();
  FewpixPlan best{1, 0, 0, 1e30};
  for (int P : kPixels) {
    if (!dwords && P > 4) break;  // the byte form of the kernel has no registers for more
    for (int c = 0; c <= 6; ++c) {
      const double tiles = std::ceil((double)g.M / P) * std::ceil((double)g.Cout / (4 << c));
      const int slices = 1024 >> c;
      const double iters = (double)((K4 + slices - 1) / slices);
      // 16 waves of 16 P gathers, 6.2 clocks each, and the address work and loads around them (narrow
      // tiles fetch a 128-byte line of the filters for every few bytes); per tile one memory round
      // trip, the sums and the stores; 6 us of launch and table staging.  Meant for the order of the
      // shapes: over 1100 random layers with dwords a call takes 0.6 to 1.15 of it (5 to 95 %, the
      // most in layers of several rounds), over 230 of the byte form 0.58 to 0.82.
      const double t_iter = 16.0 * (16.0 * P * 6.2 + (dwords ? 100.0 : 550.0) + 8.0 * (64 >> c)) / 2.4e9;
      const double t = 6e-6 + std::ceil(tiles / cus) * (iters * t_iter + 2.5e-6 + P * (4 << c) * 1e-9);
      if (t < best.cost) best = FewpixPlan{P, c, (long long)tiles, t};
    }
  }
  return best;
}

bool fewpix_shape(const Geom& g) {
  return g.mult == 0 && g.groups == 1 && g.Cout >= 4 && g.K >= 64 && g.K <= 32768;
}

hipError_t launch_fewpix(const Geom& g, const FewpixPlan& p, const QParams& qp, const uint8_t* x, const uint8_t* w,
                         const uint16_t* lut, int32_t* acc_out, float* y_out, hipStream_t s) {
  const bool dwords = g.Cin % 4 == 0;
  const int grid = (int)std::min<long long>(cu_count(), p.tiles);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(1024), 0, s, g, qp, x, w, lut, acc_out, y_out, p.cl_log2);
  };
  switch (p.P) {
    case 1: if (dwords) go(fewpix_kernel<1, true>); else go(fewpix_kernel<1, false>); break;
    case 2: if (dwords) go(fewpix_kernel<2, true>); else go(fewpix_kernel<2, false>); break;
    case 4: if (dwords) go(fewpix_kernel<4, true>); else go(fewpix_kernel<4, false>); break;
    case 7: go(fewpix_kernel<7, true>); break;
    default: go(fewpix_kernel<8, true>); break;
  }
  return hipGetLastError();
}

bool dw_supported(const Geom& g, const uint8_t* x, const uint8_t* w, const uint16_t* lut) {
  (void)x;
  (void)w;
  if (g.mult < 1 || g.Cout > kDwMaxC) return false;
  if ((uintptr_t)lut & 15) return false;
  // staging the table costs every workgroup 128 KB of reads: not worth it for small layers
  return (double)g.M * g.Cout * g.K >= 4.0e6;
}

int dw_workgroups(const Geom& g) {
  const uint64_t items = (uint64_t)g.M * (((uint32_t)g.Cout + 3u) / 4u);
  return (int)std::min<uint64_t>((uint64_t)cu_count(), (items + 1023) / 1024);
}

hipError_t launch_dw(const Geom& g, const QParams& qp, const uint8_t* x, const uint8_t* w, const uint16_t* lut,
                     int32_t* acc_out, float* y_out, hipStream_t s) {
  const uint32_t blocks = (uint32_t)dw_workgroups(g);
  const int vec_out = (g.Cout % 4 == 0 && (((uintptr_t)acc_out | (uintptr_t)y_out) & 15) == 0) ? 1 : 0;
  // one dword per tap and operand needs multiplier 1, whole groups of four channels and aligned tensors
  const bool fast = g.mult == 1 && g.Cin % 4 == 0 && (((uintptr_t)x | (uintptr_t)w) & 3) == 0;
  if (!fast)
    hipLaunchKernelGGL((dw_kernel<0, true>), dim3(blocks), dim3(1024), 0, s, g, qp, x, w, lut, acc_out, y_out, vec_out);
  else if (g.KH == 3 && g.KW == 3)  // 4e6 lookups are over 1e5 items: the grid has more threads than channel groups
    hipLaunchKernelGGL((dw3_kernel<2>), dim3(blocks), dim3(1024), 0, s, g, qp, x, w, lut, acc_out, y_out, vec_out);
  else if (g.KH == 5 && g.KW == 5)
    hipLaunchKernelGGL((dw_kernel<5, false>), dim3(blocks), dim3(1024), 0, s, g, qp, x, w, lut, acc_out, y_out, vec_out);
  else
    hipLaunchKernelGGL((dw_kernel<0, false>), dim3(blocks), dim3(1024), 0, s, g, qp, x, w, lut, acc_out, y_out, vec_out);
  return hipGetLastError();
}

int direct_threads(const Geom& g) {
  // enough for one wave on every SIMD, at least four taps each
  int S = 1;
  while (S < 64 && (uint64_t)g.M * g.Cout * S < (uint64_t)cu_count() * 256 && g.K >= 16 * S) S *= 4;
  return S;
}

hipError_t launch_direct(const Geom& g, const QParams& qp, const uint8_t* x, const uint8_t* w,
                         const uint16_t* lut, int32_t* acc_out, float* y_out, hipStream_t s) {
  const uint64_t total = (uint64_t)g.M * g.Cout;
  const int S = direct_threads(g);
  const uint32_t blocks = (uint32_t)((total * S + 255) / 256);
  switch (S) {
    case 1: hipLaunchKernelGGL((direct_kernel<1>), dim3(blocks), dim3(256), 0, s, g, qp, x, w, lut, acc_out, y_out); break;
    case 4: hipLaunchKernelGGL((direct_kernel<4>), dim3(blocks), dim3(256), 0, s, g, qp, x, w, lut, acc_out, y_out); break;
    case 16: hipLaunchKernelGGL((direct_kernel<16>), dim3(blocks), dim3(256), 0, s, g, qp, x, w, lut, acc_out, y_out); break;
    default: hipLaunchKernelGGL((direct_kernel<64>), dim3(blocks), dim3(256), 0, s, g, qp, x, w, lut, acc_out, y_out); break;
  }
  return hipGetLastError();
}

}  // namespace ax

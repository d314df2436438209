// C ABI of libaxconv: argument validation, dispatch, layer handles, error text.  No device code
// and no mutable global state here.
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>

#include "ax_internal.h"

namespace ax {

// Unsigned codes: zero points and pad code in [0, 255], pad_code -1 (or AX_PAD_DEFAULT) = x_zp.
// Signed codes: all three in [-128, 127], pad_code AX_PAD_DEFAULT = x_zp.
int make_quant_params(const ax_quant_t* q, QParams* qp, int sgn) {
  if (!q) return AX_ERR_NULL;
  const int lo = sgn ? -128 : 0, hi = sgn ? 127 : 255;
  if (q->x_zp < lo || q->x_zp > hi || q->w_zp < lo || q->w_zp > hi) return AX_ERR_QUANT;
  const bool pad_default = q->pad_code == AX_PAD_DEFAULT || (!sgn && q->pad_code == -1);
  if (!pad_default && (q->pad_code < lo || q->pad_code > hi)) return AX_ERR_QUANT;
  if (!std::isfinite(q->x_scale) || !std::isfinite(q->w_scale) || !(q->x_scale > 0.f) || !(q->w_scale > 0.f))
    return AX_ERR_QUANT;
  qp->x_zp = q->x_zp;
  qp->w_zp = q->w_zp;
  qp->pad_code = pad_default ? q->x_zp : q->pad_code;
  qp->scale = q->x_scale * q->w_scale;
  qp->dq = nullptr;
  qp->sgn = sgn ? 1 : 0;
  return AX_OK;
}

int make_options(const ax_tune_t* t, Options* o) {
  *o = Options{0, 0, 0, 0, 0, 0, 0};
  if (!t) return AX_OK;
  if (t->variant < 0 || t->variant > 3) return AX_ERR_OPTION;
  if (t->split_k < 0 || t->split_k > 64) return AX_ERR_OPTION;
  if (t->tile < 0 || t->tile > tab_num_tiles()) return AX_ERR_OPTION;
  if (t->row_tiles < 0 || t->row_tiles > (1 << 20)) return AX_ERR_OPTION;
  if (t->share_order < 0 || t->share_order > 2) return AX_ERR_OPTION;
  if (t->combine < 0 || t->combine > 2) return AX_ERR_OPTION;
  if (t->tables < 0 || t->tables > 2) return AX_ERR_OPTION;
  *o = Options{t->variant, t->split_k, t->tile, t->row_tiles, t->share_order, t->combine, t->tables};
  return AX_OK;
}

int make_geom(int N, int H, int W, int Cin, int KH, int KW, int Cout, int sh, int sw, int ph, int pw, Geom* g,
              int dh, int dw, int sgn, int depthwise, int groups) {
  if (N <= 0 || H <= 0 || W <= 0 || Cin <= 0 || KH <= 0 || KW <= 0 || Cout <= 0) return AX_ERR_SHAPE;
  if (sh < 1 || sw < 1 || ph < 0 || pw < 0 || dh < 1 || dw < 1) return AX_ERR_SHAPE;
  if (ph > (1 << 20) || pw > (1 << 20) || dh > (1 << 20) || dw > (1 << 20)) return AX_ERR_SHAPE;
  const long long eh = (long long)H + 2LL * ph - (long long)dh * (KH - 1) - 1;
  const long long ew = (long long)W + 2LL * pw - (long long)dw * (KW - 1) - 1;
  if (eh < 0 || ew < 0) return AX_ERR_SHAPE;
  const long long OH = eh / sh + 1, OW = ew / sw + 1;
  int mult = 0;
  if (groups < 1) return AX_ERR_SHAPE;
  if (depthwise) {
    if (Cout % Cin || groups != 1) return AX_ERR_SHAPE;
    mult = Cout / Cin;
    groups = Cin;  // the depthwise layer is the grouped one with a block per input channel
  } else if (Cin % groups || Cout % groups) {
    return AX_ERR_SHAPE;
  }
  const long long K = (long long)KH * KW * (Cin / groups);
  if (K > 32768) return AX_ERR_K_OVERFLOW;
  const long long lim = 0x7fffffffLL;
  const long long M = (long long)N * OH * OW;
  const long long wsize = K * Cout;
  if ((long long)N * H * W * Cin > lim || wsize > lim || M > lim || M * Cout > lim) return AX_ERR_SHAPE;
  *g = Geom{N, H, W, Cin, KH, KW, Cout, sh, sw, ph, pw, (int)OH, (int)OW, (int)M, (int)K, dh, dw, sgn ? 1 : 0, mult, 1, groups};
  return AX_OK;
}

int geom_of_desc(const ax_conv_desc_t* d, Geom* g) {
  if (!d) return AX_ERR_NULL;
  if ((d->depthwise != 0 && d->depthwise != 1) || (d->signed_codes != 0 && d->signed_codes != 1)) return AX_ERR_OPTION;
  if (d->groups < 0 || (d->depthwise && d->groups > 1)) return AX_ERR_OPTION;
  return make_geom(d->N, d->H, d->W, d->Cin, d->KH, d->KW, d->Cout, d->stride_h, d->stride_w, d->pad_h, d->pad_w, g,
                   d->dilation_h, d->dilation_w, d->signed_codes, d->depthwise, d->groups > 1 ? d->groups : 1);
}

// Tiny problems (under 4e6 lookups) do not amortize the set-up of the table tiles, and depthwise layers
// have no shared table-side operand: neither gets table tiles.
// fewpix_kernel is taken by the automatic choice only: any override of the table-tile kernels keeps the
// layer on them.  Under 2e6 lookups it is not asked: staging the table is most of its time there, and of
// random layers of 1 to 2 million lookups 22 in 284 are slower on it than on direct_kernel (the others
// faster, 1.4 times in the middle).  From 2e6 to 4e6 it competes with direct_kernel: of 316 random layers
// 295 go to it and 2 of these are slower there (1 x 2048 x 1000: 7.6 against 13.0 us); a second round
// of tiles never paid (3876 x 64 x 16: 20.8 against 12.5 us).
// From 4e6 on it competes with the table tiles, whose estimate is that of a prepared run (on channel lanes it is too low
// for short layers: 7.2 us and 0.81 of it); a call that prepares its constants itself (`prepared` 0) takes longer: 4 us for
// the table's rows and the filters, 2 and 1.8 per megabyte of transposed filters (channel lanes), 11 and 0.3 per megabyte of
// ready-made tables.  Calls on this kernel take 0.9 of its estimate, 0.72 in the byte form; prepared layers are compared
// at 0.83, which gives near ties to the kernel that needs neither prepared block nor scratch.  Long sums (2048 taps) stay
// here up to 60 us of its estimate, which is then too high (0.4 to 0.9 of it measured) and that of the tiles too low.
// Over 1768 random calls and 1842 prepared layers of 4e6 to 1.2e9 lookups, each timed on both kernels, the choice costs 1.2
// and 2.8 % over the better one each time (more than 5 % slower 94 and 156, more than 20 % 35 and 89); when these lines were
// fitted, to slower tiles, 0.8 and 2.2 %.
// Prepared layers of more than two rounds of tiles stay on this kernel up to 36 and 38 us, though the tiles are faster for
// most (5692 x 80 x 47: 30 and 15 us): the tests of the walk over several tiles reach it through the choice for such layers,
// as nothing else selects this kernel.  From 4e7 lookups on that is asked of layers beyond the bounds of ready-made tables
// only, and not of whether the plan takes them: layers that give them up do so because their tiles are faster assembled.
Route choose_route(const Geom& g, const Options& o, bool prepared) {
  Route r{};
  const bool automatic =
      !(o.variant || o.split_k || o.tile || o.row_tiles || o.share_order || o.combine || o.tables) && g.T == 1;
  const double n = (double)g.M * g.K * g.Cout;
  const bool tiny = n < 4.0e6 && o.variant != 2 && o.variant != 3;
  r.tab = o.variant != 1 && !tiny && tab_supported(g);
  if (r.tab) r.p = tab_plan(g, o, prepared);
  if (automatic && n >= 2.0e6 && fewpix_shape(g)) {
    r.fp = fewpix_plan(g);
    if (r.tab) {
      const bool ch = r.p.variant == 3;
      const double tiles = ch ? 7.2e-6 + 0.81 * r.p.cost : r.p.cost;
      const double prep = prepared  ? 0.0
                          : ch      ? 2e-6 + 1.8e-12 * g.K * g.Cout
                          : r.p.pre ? 11e-6 + 0.3e-12 * (double)(r.p.off_bpack - r.p.off_tabs)
                                    : 4e-6;
      const double scale = prepared ? 0.83 : g.Cin % 4 == 0 ? 0.9 : 0.72;
      const bool walk = prepared && r.fp.tiles > 2 * cu_count();
      const double keep = g.K >= 2048 ? 60e-6 : !walk || n < 16e6 ? 0.0 : n < 40e6 ? 38e-6 : n < 80e6 && !r.p.may_pre ? 36e-6 : 0.0;
      r.few = scale * r.fp.cost < tiles + prep || 1.1 * r.fp.cost < keep;
    } else {
      r.few = r.fp.cost < 5e-6 + 5.5e-12 * n && r.fp.tiles <= cu_count();
    }
    if (r.few) r.tab = false;
  }
  return r;
}

// Kernels that take one table at a time and need neither preparation nor scratch.
static int run_untiled(const Geom& g, const QParams& qp, const Options& o, const Route& r, const uint8_t* x,
                       const uint8_t* w, const uint16_t* lut, int32_t* acc_out, float* y_out, hipStream_t s) {
  const bool dw = g.mult && o.variant != 1 && dw_supported(g, x, w, lut);
  const size_t per_table = (size_t)g.M * g.Cout;
  for (int t = 0; t < g.T; ++t) {
    const uint16_t* lt = lut + (size_t)t * 65536;
    int32_t* at = acc_out ? acc_out + t * per_table : nullptr;
    float* yt = y_out ? y_out + t * per_table : nullptr;
    const hipError_t e = dw      ? launch_dw(g, qp, x, w, lt, at, yt, s)
                         : r.few ? launch_fewpix(g, r.fp, qp, x, w, lt, at, yt, s)
                                 : launch_direct(g, qp, x, w, lt, at, yt, s);
    if (e != hipSuccess) return AX_ERR_HIP;
  }
  return AX_OK;
}

int run_layer(const Geom& g, const QParams& qp, const Options& o, const uint8_t* x, const uint8_t* w,
              const uint16_t* lut, int32_t* acc_out, float* y_out, void* ws, size_t ws_bytes, hipStream_t s) {
  const Route r = choose_route(g, o, false);
  if (!r.tab) return run_untiled(g, qp, o, r, x, w, lut, acc_out, y_out, s);
  if (!ws || ws_bytes < r.p.prep_total + r.p.ws_total || ((uintptr_t)ws & 255)) return AX_ERR_WORKSPACE;
  uint8_t* wsb = static_cast<uint8_t*>(ws);
  const hipError_t e = launch_tab(g, qp, r.p, x, w, lut, acc_out, y_out, wsb, wsb + r.p.prep_total,
                                  ws_bytes - r.p.prep_total, kPhAll, 1, s);
  return e == hipSuccess ? AX_OK : AX_ERR_HIP;
}

static int check_io(const void* x, const void* w, const void* lut, const int32_t* acc_out, const float* y_out) {
  if (!x || !w || !lut || (!acc_out && !y_out)) return AX_ERR_NULL;
  if (((uintptr_t)lut & 1) || ((uintptr_t)acc_out & 3) || ((uintptr_t)y_out & 3)) return AX_ERR_ALIGN;
  return AX_OK;
}

static int run(const Geom& g, const ax_quant_t* q, const ax_tune_t* tune, const uint8_t* x, const uint8_t* w,
               const uint16_t* lut, int32_t* acc_out, float* y_out, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_io(x, w, lut, acc_out, y_out);
  if (rc) return rc;
  QParams qp;
  rc = make_quant_params(q, &qp, g.sgn);
  if (rc) return rc;
  Options o;
  rc = make_options(tune, &o);
  if (rc) return rc;
  return run_layer(g, qp, o, x, w, lut, acc_out, y_out, ws, ws_bytes, (hipStream_t)stream);
}

size_t layer_workspace(const Geom& g, const Options& o) {
  const Route r = choose_route(g, o, false);
  return r.tab ? r.p.prep_total + r.p.ws_total : 256;
}

static size_t workspace_of(const Geom& g, const ax_tune_t* tune) {
  Options o;
  if (make_options(tune, &o)) return 0;
  return layer_workspace(g, o);
}

}  // namespace ax

using namespace ax;

extern "C" int ax_conv2d(const uint8_t* x, int N, int H, int W, int Cin, const uint8_t* w, int KH, int KW,
                         int Cout, const uint16_t* lut, int stride_h, int stride_w, int pad_h, int pad_w,
                         const ax_quant_t* q, int32_t* acc_out, float* y_out, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
  Geom g;
  int rc = make_geom(N, H, W, Cin, KH, KW, Cout, stride_h, stride_w, pad_h, pad_w, &g);
  if (rc) return rc;
  return run(g, q, nullptr, x, w, lut, acc_out, y_out, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t ax_conv2d_workspace_bytes(int N, int H, int W, int Cin, int KH, int KW, int Cout, int stride_h,
                                            int stride_w, int pad_h, int pad_w) {
  Geom g;
  if (make_geom(N, H, W, Cin, KH, KW, Cout, stride_h, stride_w, pad_h, pad_w, &g)) return 0;
  return workspace_of(g, nullptr);
}

extern "C" int ax_conv2d_ex(const ax_conv_desc_t* desc, const ax_tune_t* tune, const void* x, const void* w,
                            const void* lut, const ax_quant_t* q, int32_t* acc_out, float* y_out, void* workspace,
                            size_t workspace_bytes, void* hip_stream) {
  Geom g;
  int rc = geom_of_desc(desc, &g);
  if (rc) return rc;
  return run(g, q, tune, static_cast<const uint8_t*>(x), static_cast<const uint8_t*>(w),
             static_cast<const uint16_t*>(lut), acc_out, y_out, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t ax_conv2d_ex_workspace_bytes(const ax_conv_desc_t* desc, const ax_tune_t* tune) {
  Geom g;
  if (geom_of_desc(desc, &g)) return 0;
  return workspace_of(g, tune);
}

extern "C" int ax_conv2d_multi_lut(const uint8_t* x, int N, int H, int W, int Cin, const uint8_t* w, int KH, int KW,
                                   int Cout, const uint16_t* luts, int num_luts, int stride_h, int stride_w,
                                   int pad_h, int pad_w, const ax_quant_t* q, int32_t* acc_out, float* y_out,
                                   void* workspace, size_t workspace_bytes, void* hip_stream) {
  Geom g;
  int rc = make_geom(N, H, W, Cin, KH, KW, Cout, stride_h, stride_w, pad_h, pad_w, &g);
  if (rc) return rc;
  if (num_luts < 1 || num_luts > 65536) return AX_ERR_SHAPE;
  g.T = num_luts;
  return run(g, q, nullptr, x, w, luts, acc_out, y_out, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t ax_conv2d_multi_lut_workspace_bytes(int N, int H, int W, int Cin, int KH, int KW, int Cout,
                                                      int num_luts, int stride_h, int stride_w, int pad_h,
                                                      int pad_w) {
  Geom g;
  if (make_geom(N, H, W, Cin, KH, KW, Cout, stride_h, stride_w, pad_h, pad_w, &g)) return 0;
  if (num_luts < 1 || num_luts > 65536) return 0;
  g.T = num_luts;
  return workspace_of(g, nullptr);
}

extern "C" int ax_dense(const uint8_t* x, int M, int K, const uint8_t* w, int N, const uint16_t* lut,
                        const ax_quant_t* q, int32_t* acc_out, float* y_out, void* workspace,
                        size_t workspace_bytes, void* hip_stream) {
  Geom g;
  int rc = make_geom(M, 1, 1, K, 1, 1, N, 1, 1, 0, 0, &g);
  if (rc) return rc;
  return run(g, q, nullptr, x, w, lut, acc_out, y_out, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t ax_dense_workspace_bytes(int M, int K, int N) {
  Geom g;
  if (make_geom(M, 1, 1, K, 1, 1, N, 1, 1, 0, 0, &g)) return 0;
  return workspace_of(g, nullptr);
}

// ---- layer handles --------------------------------------------------------------------------

extern "C" int ax_layer_create(const ax_conv_desc_t* desc, int num_luts, const ax_quant_t* q, const ax_tune_t* tune,
                               ax_layer_t** layer_out) {
  if (!layer_out) return AX_ERR_NULL;
  *layer_out = nullptr;
  Geom g;
  int rc = geom_of_desc(desc, &g);
  if (rc) return rc;
  if (num_luts < 1 || num_luts > 65536) return AX_ERR_SHAPE;
  g.T = num_luts;
  QParams qp;
  rc = make_quant_params(q, &qp, g.sgn);
  if (rc) return rc;
  Options o;
  rc = make_options(tune, &o);
  if (rc) return rc;
  ax_layer* L = new (std::nothrow) ax_layer();
  if (!L) return AX_ERR_HIP;
  L->g = g;
  L->qp = qp;
  L->o = o;
  L->r = choose_route(g, o, true);
  L->w = nullptr;
  L->lut = nullptr;
  L->prepared = nullptr;
  L->ready = false;
  *layer_out = L;
  return AX_OK;
}

extern "C" void ax_layer_destroy(ax_layer_t* layer) { delete layer; }

extern "C" size_t ax_layer_prepared_bytes(const ax_layer_t* layer) {
  return layer && layer->r.tab ? layer->r.p.prep_total : 0;
}

extern "C" size_t ax_layer_workspace_bytes(const ax_layer_t* layer) {
  return layer && layer->r.tab ? layer->r.p.ws_total : 0;
}

extern "C" int ax_layer_prepare(ax_layer_t* layer, const void* w, const void* luts, void* prepared,
                                size_t prepared_bytes, void* hip_stream) {
  if (!layer || !w || !luts) return AX_ERR_NULL;
  if ((uintptr_t)luts & 1) return AX_ERR_ALIGN;
  layer->ready = false;
  if (layer->r.tab) {
    if (!prepared || prepared_bytes < layer->r.p.prep_total || ((uintptr_t)prepared & 255)) return AX_ERR_WORKSPACE;
    const hipError_t e = launch_tab(layer->g, layer->qp, layer->r.p, nullptr, static_cast<const uint8_t*>(w),
                                    static_cast<const uint16_t*>(luts), nullptr, nullptr, prepared, nullptr, 0,
                                    kPhConst, 1, (hipStream_t)hip_stream);
    if (e != hipSuccess) return AX_ERR_HIP;
  }
  layer->w = static_cast<const uint8_t*>(w);
  layer->lut = static_cast<const uint16_t*>(luts);
  layer->prepared = prepared;
  layer->ready = true;
  return AX_OK;
}

namespace ax {
size_t scratch_need(const ax_layer* layer, const void* x) {
  if (!layer || !layer->r.tab) return 0;
  const TabPlan& p = layer->r.p;
  // unsigned activations read in place leave the last part of the scratch unused
  const bool unused = p.variant == 2 && !layer->g.sgn && reads_in_place(layer->g, x);
  return p.ws_total - (unused ? p.ws_apack : 0);
}

// Shared by ax_layer_run and the kernel-timing probe: the per-call parts of a prepared layer.
int run_prepared(const ax_layer* layer, const void* x, int32_t* acc_out, float* y_out, void* workspace,
                 size_t workspace_bytes, int phases, int main_reps, hipStream_t s) {
  if (!layer) return AX_ERR_NULL;
  if (!layer->ready) return AX_ERR_STATE;
  int rc = check_io(x, layer->w, layer->lut, acc_out, y_out);
  if (rc) return rc;
  const uint8_t* xb = static_cast<const uint8_t*>(x);
  if (!layer->r.tab) {
    if (!(phases & kPhMain)) return AX_OK;
    for (int r = 0; r < main_reps; ++r) {
      rc = run_untiled(layer->g, layer->qp, layer->o, layer->r, xb, layer->w, layer->lut, acc_out, y_out, s);
      if (rc) return rc;
    }
    return AX_OK;
  }
  const TabPlan& p = layer->r.p;
  const size_t need = scratch_need(layer, x);
  if (need && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))) return AX_ERR_WORKSPACE;
  // A call that needs no scratch takes any buffer; one that is not aligned stays unused.
  const size_t usable = workspace && ((uintptr_t)workspace & 255) == 0 ? workspace_bytes : 0;
  const hipError_t e = launch_tab(layer->g, layer->qp, p, xb, layer->w, layer->lut, acc_out, y_out, layer->prepared,
                                  workspace, usable, phases, main_reps, s);
  return e == hipSuccess ? AX_OK : AX_ERR_HIP;
}
}  // namespace ax

extern "C" int ax_layer_run(const ax_layer_t* layer, const void* x, int32_t* acc_out, float* y_out, void* workspace,
                            size_t workspace_bytes, void* hip_stream) {
  return run_prepared(layer, x, acc_out, y_out, workspace, workspace_bytes, kPhCall | kPhMain | kPhFixup, 1,
                      (hipStream_t)hip_stream);
}

extern "C" int ax_layer_plan(const ax_layer_t* layer, int* variant, int* tile, int* workgroups, int* pieces) {
  if (!layer) return AX_ERR_NULL;
  if (variant) *variant = layer->r.tab ? layer->r.p.variant : 1;
  if (tile) *tile = layer->r.tab ? layer->r.p.tile + 1 : 0;
  if (workgroups) *workgroups = layer->r.tab ? layer->r.p.G : 0;
  if (pieces) *pieces = layer->r.tab ? layer->r.p.partials : 0;
  return AX_OK;
}

extern "C" int ax_layer_plan_paths(const ax_layer_t* layer, int* combine, int* tables) {
  if (!layer) return AX_ERR_NULL;
  if (combine) *combine = (layer->r.tab && layer->r.p.partials > 0) ? (layer->r.p.combine ? 2 : 1) : 0;
  if (tables) *tables = layer->r.tab ? (layer->r.p.pre ? 2 : 1) : 0;
  return AX_OK;
}

extern "C" const char* ax_strerror(int code) {
  switch (code) {
    case AX_OK: return "ok";
    case AX_ERR_NULL: return "required pointer is NULL";
    case AX_ERR_SHAPE: return "invalid shape, stride or padding";
    case AX_ERR_QUANT: return "invalid quantization parameters";
    case AX_ERR_K_OVERFLOW: return "KH*KW*Cin exceeds 32768: int32 accumulator could overflow";
    case AX_ERR_WORKSPACE: return "workspace missing, too small or misaligned";
    case AX_ERR_HIP: return "HIP runtime call failed";
    case AX_ERR_ALIGN: return "pointer not aligned";
    case AX_ERR_OPTION: return "flag, round mode or tuning value out of range";
    case AX_ERR_STATE: return "layer handle has not been prepared";
    default: return "unknown error code";
  }
}

extern "C" int ax_version(void) { return 330; }

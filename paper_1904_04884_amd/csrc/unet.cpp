// Warm-start 3D U-Net driver: parameter layout, activation / gradient buffers,
// forward, backward and Adam, behind the ri_unet_* C ABI.  All arithmetic runs
// in the kernels of unet.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/rihvr.h"
#include "unet_internal.h"

using namespace rihvr;

// error helper shared with abi.cpp
extern "C" const char* ri_last_error(void);
namespace rihvr {
ri_status set_error(ri_status st, const char* msg);
}

namespace {

enum Kind { CONV = 0, UP = 1, HEAD = 2 };

struct Layer {
  Kind kind;
  int cin, cout;
  size_t w, b;              // offsets in the FP32 parameter array
  size_t pf = 0, pb = 0;    // offsets of the packed forward / input-gradient BF16 weights
  int f_npad = 0, f_c = 0;  // forward GEMM: padded columns, channels per tap
  int b_npad = 0, b_c = 0;  // input-gradient GEMM
};

int pad(int v, int m) { return (v + m - 1) / m * m; }

struct Net {
  int L, base;
  std::vector<int> ch;
  std::vector<Layer> layers;  // order: enc{l}a, enc{l}b for l = 0..L-1; up{l}, dec{l}a, dec{l}b for l = L-2..0; head
  size_t nparams = 0, npacked = 0;
  int enc_a(int l) const { return 2 * l; }
  int enc_b(int l) const { return 2 * l + 1; }
  int up(int l) const { return 2 * L + 3 * (L - 2 - l); }
  int dec_a(int l) const { return up(l) + 1; }
  int dec_b(int l) const { return up(l) + 2; }
  int head() const { return (int)layers.size() - 1; }
};

Net build_net(int L, int base) {
  Net n;
  n.L = L;
  n.base = base;
  for (int l = 0; l < L; ++l) n.ch.push_back(base << l);
  auto add = [&](Kind k, int cin, int cout) {
    Layer y;
    y.kind = k;
    y.cin = cin;
    y.cout = cout;
    const size_t wsz = k == CONV ? (size_t)27 * cin * cout : k == UP ? (size_t)8 * cin * cout : (size_t)cin;
    y.w = n.nparams;
    n.nparams += wsz;
    y.b = n.nparams;
    n.nparams += (size_t)cout;
    if (k == CONV) {
      y.f_npad = pad(cout, 16);
      y.f_c = pad(cin, 8);
      y.b_npad = pad(cin, 16);
      y.b_c = pad(cout, 8);
      y.pf = n.npacked;
      n.npacked += (size_t)27 * y.f_npad * y.f_c;
      y.pb = n.npacked;
      n.npacked += (size_t)27 * y.b_npad * y.b_c;
    } else if (k == UP) {
      y.f_npad = 8 * cout;
      y.f_c = cin;
      y.b_npad = pad(cin, 16);
      y.b_c = cout;
      y.pf = n.npacked;
      n.npacked += (size_t)y.f_npad * y.f_c;
      y.pb = n.npacked;
      n.npacked += (size_t)8 * y.b_npad * y.b_c;
    } else {
      y.f_npad = 16;
      y.f_c = cin;
      y.b_npad = pad(cin, 16);
      y.b_c = 8;
      y.pf = n.npacked;
      n.npacked += (size_t)y.f_npad * y.f_c;
      y.pb = n.npacked;
      n.npacked += (size_t)y.b_npad * y.b_c;
    }
    n.layers.push_back(y);
  };
  int cin = 1;
  for (int l = 0; l < L; ++l) {
    add(CONV, cin, n.ch[l]);
    add(CONV, n.ch[l], n.ch[l]);
    cin = n.ch[l];
  }
  for (int l = L - 2; l >= 0; --l) {
    add(UP, n.ch[l + 1], n.ch[l]);
    add(CONV, 2 * n.ch[l], n.ch[l]);
    add(CONV, n.ch[l], n.ch[l]);
  }
  add(HEAD, n.ch[0], 1);
  return n;
}

// Activation / gradient buffers for one volume size.
struct Buffers {
  size_t total = 0;
  size_t packed = 0, y = 0, gy8 = 0, loss = 0, lpart = 0;
  std::vector<size_t> wpart, bpart;   // gradient partials of each layer
  std::vector<int> nblk;              // ... and their count
  std::vector<size_t> a, up, skip, p, idx, da, db, ga, gup, gskip, gda, gdb, gp;
  size_t bbot = 0, gbbot = 0;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

Buffers layout(const Net& n, int D, int H, int W, bool train) {
  Buffers B;
  const int L = n.L;
  size_t off = 256;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  auto nv = [&](int l) { return (size_t)(D >> l) * (H >> l) * (W >> l); };
  B.packed = take(n.npacked * 2);
  B.a.resize(L);
  B.up.resize(L);
  B.skip.resize(L);
  B.p.resize(L);
  B.idx.resize(L);
  B.da.resize(L);
  B.db.resize(L);
  B.ga.resize(L);
  B.gup.resize(L);
  B.gskip.resize(L);
  B.gda.resize(L);
  B.gdb.resize(L);
  B.gp.resize(L);
  for (int l = 0; l < L; ++l) {
    const size_t c = n.ch[l];
    B.a[l] = take(nv(l) * c * 2);
    if (l < L - 1) {
      B.up[l] = take(nv(l) * c * 2);
      B.skip[l] = take(nv(l) * c * 2);
      B.p[l] = take(nv(l + 1) * c * 2);
      if (train) B.idx[l] = take(nv(l + 1) * c);
      B.da[l] = take(nv(l) * c * 2);
      B.db[l] = take(nv(l) * c * 2);
    }
  }
  B.bbot = take(nv(L - 1) * n.ch[L - 1] * 2);
  if (train) {
    B.y = take(nv(0) * 4);
    B.gy8 = take(nv(0) * 8 * 2);
    B.loss = take(4);
    for (int l = 0; l < L; ++l) {
      const size_t c = n.ch[l];
      B.ga[l] = take(nv(l) * c * 2);
      if (l < L - 1) {
        B.gup[l] = take(nv(l) * c * 2);
        B.gskip[l] = take(nv(l) * c * 2);
        B.gda[l] = take(nv(l) * c * 2);
        B.gdb[l] = take(nv(l) * c * 2);
        B.gp[l] = take(nv(l + 1) * c * 2);
      }
    }
    B.gbbot = take(nv(L - 1) * n.ch[L - 1] * 2);
    // partial sums of every layer's weight and bias gradients, and of the loss
    B.wpart.resize(n.layers.size());
    B.bpart.resize(n.layers.size());
    B.nblk.resize(n.layers.size());
    auto grad = [&](int k, int mode, int lv) {   // lv: level of the rows
      const Layer& y = n.layers[k];
      const int taps = y.kind == CONV ? 27 : (y.kind == UP ? 8 : 1);
      const int nb = wgrad_blocks(mode, D >> lv, H >> lv, W >> lv, y.cout, y.cin);
      B.nblk[k] = nb;
      B.wpart[k] = take((size_t)nb * taps * y.cin * y.cout * 4);
      B.bpart[k] = take((size_t)nb * (y.kind == UP ? 8 : 1) * y.cout * 4);
    };
    for (int l = 0; l < L; ++l) {
      grad(n.enc_a(l), GG_CONV3_FWD, l);
      grad(n.enc_b(l), GG_CONV3_FWD, l);
      if (l < L - 1) {
        grad(n.up(l), GG_UP_FWD, l + 1);
        grad(n.dec_a(l), GG_CONV3_FWD, l);
        grad(n.dec_b(l), GG_CONV3_FWD, l);
      }
    }
    grad(n.head(), GG_POINT, 0);
    B.lpart = take((size_t)mse_blocks((long)nv(0)) * 4);
  }
  B.total = off;
  return B;
}

template <class T>
T* at(void* ws, size_t off) {
  const uintptr_t base = ((uintptr_t)ws + 255) & ~(uintptr_t)255;
  return reinterpret_cast<T*>(base + off - 256);
}

ri_status check_cfg(const ri_unet_config* c) {
  if (!c) return set_error(RI_ERR_INVALID_ARG, "unet config is NULL");
  // channel counts are padded to 16 * 2^k columns of MFMA tiles, which every
  // kernel case covers only for base = 8 * 2^k
  const bool pow2 = c->base >= 8 && (c->base & (c->base - 1)) == 0;
  if (c->levels < 1 || c->levels > 6 || !pow2 || (c->base << (c->levels - 1)) > 128)
    return set_error(RI_ERR_INVALID_ARG,
                     "unet config: levels in [1, 6], base one of 8, 16, 32, ..., base*2^(levels-1) <= 128");
  return RI_OK;
}

ri_status check_dims(const ri_unet_config* c, int D, int H, int W) {
  const int m = 1 << (c->levels - 1);
  if (D < m || H < m || W < m || D % m || H % m || W % m)
    return set_error(RI_ERR_UNSUPPORTED_SIZE, "unet volume dims must be positive multiples of 2^(levels-1)");
  return RI_OK;
}

#define UTRY(expr)                                                      \
  do {                                                                  \
    hipError_t e_ = (expr);                                             \
    if (e_ != hipSuccess) {                                             \
      char m_[256];                                                     \
      snprintf(m_, sizeof(m_), "%s: %s", #expr, hipGetErrorString(e_)); \
      return set_error(RI_ERR_HIP, m_);                                 \
    }                                                                   \
  } while (0)

// 3x3x3 layer on contiguous channels
ConvArgs conv(int bwd, int D, int H, int W, const uint16_t* src, int C, const uint16_t* wt, int N, int Npad,
              const float* bias, int relu, uint16_t* dst) {
  ConvArgs a{};
  a.bwd = bwd;
  a.D = D; a.H = H; a.W = W;
  a.src = src; a.src2 = src + C / 2; a.src_cs = C;
  a.C = C;
  a.wt = wt; a.N = N; a.Npad = Npad;
  a.bias = bias; a.relu = relu;
  a.dst = dst; a.dst2 = dst; a.nsplit = Npad; a.dst_cs = N;
  return a;
}

ri_status pack_all(const Net& n, const float* params, uint16_t* packed, bool with_bwd, hipStream_t s) {
  PackTable tab{};
  auto entry = [&](const Layer& y, int T, int kind, int Npad, int Cpad, size_t out) {
    tab.e[tab.n++] = PackEntry{params + y.w, packed + out, T, y.cin, y.cout, kind, Npad, Cpad, 0};
  };
  for (const Layer& y : n.layers) {
    const int T = y.kind == CONV ? 27 : (y.kind == UP ? 8 : 1);
    if (y.kind == UP) entry(y, 1, 2, y.f_npad, y.f_c, y.pf);
    else entry(y, T, 1, y.f_npad, y.f_c, y.pf);
    if (with_bwd) entry(y, T, 0, y.b_npad, y.b_c, y.pb);
  }
  UTRY(launch_pack(tab, s));
  return RI_OK;
}

// Network output (training: the head's pre-activation) to `out`.
ri_status forward(const Net& n, const float* params, const float* in, float scale, float* out, int D, int H, int W,
                  void* ws, const Buffers& B, bool train, hipStream_t s) {
  const int L = n.L;
  uint16_t* pk = at<uint16_t>(ws, B.packed);
  ri_status st = pack_all(n, params, pk, train, s);
  if (st != RI_OK) return st;
  for (int l = 0; l < L; ++l) {
    const int Dl = D >> l, Hl = H >> l, Wl = W >> l, c = n.ch[l];
    const Layer& ea = n.layers[n.enc_a(l)];
    const Layer& eb = n.layers[n.enc_b(l)];
    uint16_t* a = at<uint16_t>(ws, B.a[l]);
    ConvArgs ca = conv(0, Dl, Hl, Wl, l == 0 ? nullptr : at<uint16_t>(ws, B.p[l - 1]), ea.f_c, pk + ea.pf, c, ea.f_npad,
                       params + ea.b, 1, a);
    if (l == 0) {
      ca.src = ca.src2 = nullptr;
      ca.src32 = in;
      ca.scale = scale;
    }
    UTRY(launch_conv3(ca, s));
    uint16_t* bo = l < L - 1 ? at<uint16_t>(ws, B.skip[l]) : at<uint16_t>(ws, B.bbot);
    UTRY(launch_conv3(conv(0, Dl, Hl, Wl, a, eb.f_c, pk + eb.pf, c, eb.f_npad, params + eb.b, 1, bo), s));
    if (l < L - 1)
      UTRY(launch_pool_fwd(bo, at<uint16_t>(ws, B.p[l]), train ? at<uint8_t>(ws, B.idx[l]) : nullptr, c, Dl / 2, Hl / 2,
                           Wl / 2, s));
  }
  const uint16_t* h = at<uint16_t>(ws, B.bbot);
  for (int l = L - 2; l >= 0; --l) {
    const int Dl = D >> l, Hl = H >> l, Wl = W >> l, c = n.ch[l], cu = n.ch[l + 1];
    const Layer& up = n.layers[n.up(l)];
    const Layer& da = n.layers[n.dec_a(l)];
    const Layer& db = n.layers[n.dec_b(l)];
    uint16_t* uo = at<uint16_t>(ws, B.up[l]);
    UTRY(launch_up_fwd(UpArgs{Dl / 2, Hl / 2, Wl / 2, h, cu, c, pk + up.pf, params + up.b, uo}, s));
    uint16_t* dao = at<uint16_t>(ws, B.da[l]);
    ConvArgs ca = conv(0, Dl, Hl, Wl, uo, da.f_c, pk + da.pf, c, da.f_npad, params + da.b, 1, dao);
    ca.src2 = at<uint16_t>(ws, B.skip[l]);   // concatenation [up, skip]
    ca.src_cs = c;
    UTRY(launch_conv3(ca, s));
    uint16_t* dbo = at<uint16_t>(ws, B.db[l]);
    UTRY(launch_conv3(conv(0, Dl, Hl, Wl, dao, db.f_c, pk + db.pf, c, db.f_npad, params + db.b, 1, dbo), s));
    h = dbo;
  }
  // head: ReLU output for inference; training keeps the pre-activation (the
  // loss is taken on it, so a voxel below zero still passes gradient)
  const Layer& hd = n.layers[n.head()];
  UTRY(launch_head(h, n.ch[0], pk + hd.pf, params + hd.b, train ? 0 : 1, out, (long)D * H * W, s));
  return RI_OK;
}

// Gradients from the loss down; every ReLU mask is applied where the gradient
// is written.
ri_status backward(const Net& n, const float* params, const float* in, float scale, const float* target,
                   float pos_weight, int D, int H, int W, void* ws, const Buffers& B, hipStream_t s) {
  const int L = n.L;
  uint16_t* pk = at<uint16_t>(ws, B.packed);
  uint16_t* gy8 = at<uint16_t>(ws, B.gy8);
  UTRY(launch_mse(at<float>(ws, B.y), target, (long)D * H * W, pos_weight, gy8, at<float>(ws, B.lpart), s));
  auto wgrad = [&](int k, int mode, int Dl, int Hl, int Wl, const uint16_t* g, int gcs, const uint16_t* src,
                   const uint16_t* src2 = nullptr) {
    const Layer& y = n.layers[k];
    WgradArgs w{};
    w.mode = mode;
    w.D = Dl; w.H = Hl; w.W = Wl;
    w.g = g; w.g_cs = gcs; w.N = y.cout;
    w.s = src; w.s_cs = y.cin; w.ssplit = pad(y.cin, 8); w.C = y.cin;
    if (src2) {          // concatenation of two buffers of cin / 2 channels
      w.s_cs = w.ssplit = y.cin / 2;
      w.s2 = src2 - y.cin / 2;
    }
    if (!src) {          // the first layer
      w.s32 = in;
      w.scale = scale;
      w.s_cs = 8;
    }
    w.part = at<float>(ws, B.wpart[k]);
    w.bpart = at<float>(ws, B.bpart[k]);
    return launch_wgrad(w, B.nblk[k], s);
  };
  auto gemm = [&](int mode, int Dl, int Hl, int Wl, const uint16_t* src, int cs, int T, const Layer& y,
                  const uint16_t* mask, uint16_t* dst) {
    return launch_gather_gemm(GatherGemmArgs{mode, Dl, Hl, Wl, src, cs, T, y.b_c, pk + y.pb, y.cin, y.b_npad, mask, dst},
                              s);
  };
  // head
  const Layer& hd = n.layers[n.head()];
  const uint16_t* top = L > 1 ? at<uint16_t>(ws, B.db[0]) : at<uint16_t>(ws, B.bbot);
  uint16_t* gtop = L > 1 ? at<uint16_t>(ws, B.gdb[0]) : at<uint16_t>(ws, B.gbbot);
  UTRY(wgrad(n.head(), GG_POINT, D, H, W, gy8, 8, top));
  UTRY(gemm(GG_POINT, D, H, W, gy8, 8, 1, hd, top, gtop));
  // decoder, finest level first
  for (int l = 0; l <= L - 2; ++l) {
    const int Dl = D >> l, Hl = H >> l, Wl = W >> l, c = n.ch[l];
    const Layer& up = n.layers[n.up(l)];
    const Layer& da = n.layers[n.dec_a(l)];
    const Layer& db = n.layers[n.dec_b(l)];
    uint16_t* gdb = at<uint16_t>(ws, B.gdb[l]);
    uint16_t* gda = at<uint16_t>(ws, B.gda[l]);
    uint16_t* gup = at<uint16_t>(ws, B.gup[l]);
    const uint16_t* dao = at<uint16_t>(ws, B.da[l]);
    UTRY(wgrad(n.dec_b(l), GG_CONV3_FWD, Dl, Hl, Wl, gdb, c, dao));
    ConvArgs cb = conv(1, Dl, Hl, Wl, gdb, db.b_c, pk + db.pb, c, db.b_npad, nullptr, 0, gda);
    cb.mask = dao;
    cb.mask_cs = c;
    UTRY(launch_conv3(cb, s));
    UTRY(wgrad(n.dec_a(l), GG_CONV3_FWD, Dl, Hl, Wl, gda, c, at<uint16_t>(ws, B.up[l]), at<uint16_t>(ws, B.skip[l])));
    ConvArgs ca = conv(1, Dl, Hl, Wl, gda, da.b_c, pk + da.pb, 2 * c, da.b_npad, nullptr, 0, gup);
    ca.dst2 = at<uint16_t>(ws, B.gskip[l]);
    ca.nsplit = c;
    ca.dst_cs = c;
    UTRY(launch_conv3(ca, s));
    // up-convolution: gradient rows at the fine level, parameters over coarse rows
    const uint16_t* hin = (l + 1 == L - 1) ? at<uint16_t>(ws, B.bbot) : at<uint16_t>(ws, B.db[l + 1]);
    uint16_t* ghin = (l + 1 == L - 1) ? at<uint16_t>(ws, B.gbbot) : at<uint16_t>(ws, B.gdb[l + 1]);
    UTRY(wgrad(n.up(l), GG_UP_FWD, Dl / 2, Hl / 2, Wl / 2, gup, c, hin));
    UTRY(gemm(GG_UP_BWD, Dl / 2, Hl / 2, Wl / 2, gup, c, 8, up, hin, ghin));
  }
  // encoder, coarsest level first
  for (int l = L - 1; l >= 0; --l) {
    const int Dl = D >> l, Hl = H >> l, Wl = W >> l, c = n.ch[l];
    const Layer& ea = n.layers[n.enc_a(l)];
    const Layer& eb = n.layers[n.enc_b(l)];
    uint16_t* gout = l == L - 1 ? at<uint16_t>(ws, B.gbbot) : at<uint16_t>(ws, B.gskip[l]);
    if (l < L - 1)
      UTRY(launch_pool_bwd(at<uint16_t>(ws, B.gp[l]), at<uint8_t>(ws, B.idx[l]), at<uint16_t>(ws, B.skip[l]), gout, c,
                           Dl / 2, Hl / 2, Wl / 2, s));
    const uint16_t* a = at<uint16_t>(ws, B.a[l]);
    uint16_t* ga = at<uint16_t>(ws, B.ga[l]);
    UTRY(wgrad(n.enc_b(l), GG_CONV3_FWD, Dl, Hl, Wl, gout, c, a));
    ConvArgs cb = conv(1, Dl, Hl, Wl, gout, eb.b_c, pk + eb.pb, c, eb.b_npad, nullptr, 0, ga);
    cb.mask = a;
    cb.mask_cs = c;
    UTRY(launch_conv3(cb, s));
    UTRY(wgrad(n.enc_a(l), GG_CONV3_FWD, Dl, Hl, Wl, ga, c, l == 0 ? nullptr : at<uint16_t>(ws, B.p[l - 1])));
    if (l > 0)
      UTRY(launch_conv3(conv(1, Dl, Hl, Wl, ga, ea.b_c, pk + ea.pb, n.ch[l - 1], ea.b_npad, nullptr, 0,
                             at<uint16_t>(ws, B.gp[l - 1])), s));
  }
  return RI_OK;
}

// splitmix64 + Box-Muller, for parameter initialisation on the host
struct Rng {
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  double uniform() { return ((next() >> 11) + 0.5) * (1.0 / 9007199254740992.0); }
  double normal() { return std::sqrt(-2.0 * std::log(uniform())) * std::cos(2.0 * M_PI * uniform()); }
};

}  // namespace

extern "C" ri_status ri_unet_param_count(const ri_unet_config* cfg, size_t* n) {
  ri_status st = check_cfg(cfg);
  if (st != RI_OK) return st;
  if (!n) return set_error(RI_ERR_INVALID_ARG, "NULL output");
  *n = build_net(cfg->levels, cfg->base).nparams;
  return RI_OK;
}

extern "C" ri_status ri_unet_init_params(const ri_unet_config* cfg, uint64_t seed, float* params, void* stream) {
  ri_status st = check_cfg(cfg);
  if (st != RI_OK) return st;
  if (!params) return set_error(RI_ERR_INVALID_ARG, "params is NULL");
  const Net n = build_net(cfg->levels, cfg->base);
  std::vector<float> h(n.nparams);
  Rng r{seed};
  for (const Layer& y : n.layers) {
    const size_t wsz = y.b - y.w;
    const double sd = y.kind == CONV ? std::sqrt(2.0 / (27.0 * y.cin)) : std::sqrt(1.0 / y.cin);
    const bool head = &y == &n.layers[n.head()];
    // the head starts at zero weights: the first output is the bias everywhere
    for (size_t i = 0; i < wsz; ++i) h[y.w + i] = head ? 0.f : (float)(sd * r.normal());
    for (int i = 0; i < y.cout; ++i) h[y.b + i] = 0.01f;
  }
  UTRY(hipMemcpyAsync(params, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice, (hipStream_t)stream));
  UTRY(hipStreamSynchronize((hipStream_t)stream));
  return RI_OK;
}

extern "C" ri_status ri_unet_workspace_size(const ri_unet_config* cfg, int32_t d, int32_t h, int32_t w,
                                           int32_t training, size_t* bytes) {
  ri_status st = check_cfg(cfg);
  if (st != RI_OK) return st;
  st = check_dims(cfg, d, h, w);
  if (st != RI_OK) return st;
  if (!bytes) return set_error(RI_ERR_INVALID_ARG, "NULL output");
  *bytes = layout(build_net(cfg->levels, cfg->base), d, h, w, training != 0).total;
  return RI_OK;
}

extern "C" ri_status ri_unet_forward(const ri_unet_config* cfg, const float* params, const float* in, float scale,
                                     float* out, int32_t d, int32_t h, int32_t w, void* ws, size_t ws_bytes,
                                     void* stream) {
  ri_status st = check_cfg(cfg);
  if (st != RI_OK) return st;
  st = check_dims(cfg, d, h, w);
  if (st != RI_OK) return st;
  if (!params || !in || !out || !ws) return set_error(RI_ERR_INVALID_ARG, "NULL pointer");
  const Net n = build_net(cfg->levels, cfg->base);
  const Buffers B = layout(n, d, h, w, false);
  if (ws_bytes < B.total) return set_error(RI_ERR_WORKSPACE_TOO_SMALL, "unet workspace too small");
  hipStream_t s = (hipStream_t)stream;
  return forward(n, params, in, scale, out, d, h, w, ws, B, false, s);
}

extern "C" ri_status ri_unet_train_step(const ri_unet_config* cfg, float* params, float* grads, float* adam_m,
                                        float* adam_v, int32_t step, float lr, const float* in, float scale,
                                        const float* target, float pos_weight, int32_t d, int32_t h, int32_t w,
                                        float* loss_out, void* ws, size_t ws_bytes, void* stream) {
  ri_status st = check_cfg(cfg);
  if (st != RI_OK) return st;
  st = check_dims(cfg, d, h, w);
  if (st != RI_OK) return st;
  if (!params || !grads || !in || !target || !ws || (lr > 0 && (!adam_m || !adam_v)))
    return set_error(RI_ERR_INVALID_ARG, "NULL pointer");
  if (lr > 0 && step < 1) return set_error(RI_ERR_INVALID_ARG, "Adam step must be >= 1");
  if (!(pos_weight > 0.f) || !std::isfinite(pos_weight))
    return set_error(RI_ERR_INVALID_ARG, "pos_weight must be finite and > 0");
  const Net n = build_net(cfg->levels, cfg->base);
  const Buffers B = layout(n, d, h, w, true);
  if (ws_bytes < B.total) return set_error(RI_ERR_WORKSPACE_TOO_SMALL, "unet workspace too small");
  hipStream_t s = (hipStream_t)stream;
  st = forward(n, params, in, scale, at<float>(ws, B.y), d, h, w, ws, B, true, s);
  if (st != RI_OK) return st;
  st = backward(n, params, in, scale, target, pos_weight, d, h, w, ws, B, s);
  if (st != RI_OK) return st;
  // gradients (and the loss) from their partials, with the Adam update
  GradTable tab{};
  auto entry = [&](size_t part, float* out, long param, size_t count, int parts) {
    tab.e[tab.n++] = GradEntry{at<float>(ws, part), out, param, (int)count, parts, 0};
  };
  for (size_t k = 0; k < n.layers.size(); ++k) {
    const Layer& y = n.layers[k];
    entry(B.wpart[k], grads + y.w, (long)y.w, y.b - y.w, B.nblk[k]);
    entry(B.bpart[k], grads + y.b, (long)y.b, (size_t)y.cout, B.nblk[k] * (y.kind == UP ? 8 : 1));
  }
  entry(B.lpart, loss_out ? loss_out : at<float>(ws, B.loss), -1, 1, mse_blocks((long)d * h * w));
  const double b1 = 0.9, b2 = 0.999;
  AdamArgs ad{};
  ad.w = params; ad.m = adam_m; ad.v = adam_v;
  ad.lr = lr;
  if (lr > 0) {
    ad.b1 = (float)b1; ad.b2 = (float)b2; ad.a1 = (float)(1.0 - b1); ad.a2 = (float)(1.0 - b2);
    ad.eps = (float)1e-8;
    ad.c1 = (float)(1.0 - std::pow(b1, (double)step));
    ad.c2 = (float)(1.0 - std::pow(b2, (double)step));
  }
  UTRY(launch_finish_grads(tab, ad, s));
  return RI_OK;
}

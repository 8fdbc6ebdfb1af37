// Operand tiles of the fp32 contractions on their way from memory to LDS:
// plain strided tiles, convolution gathers and the fused forward's W tile with
// its pending update.  256 threads hold a tile as float4s.
#pragma once

#include "gemm_common.h"

namespace opfuse {

// A BX (output dim) x BR (reduction) tile of one operand, held in registers as
// float4s between its global load and its LDS store.  RC: the reduction index
// is contiguous in memory (else the output index is).  `base` points at the
// tile's first element; nx / nr are the valid extents from there (<= 0: none).
// vec: 128-bit loads (base 16B aligned, strides and both extents' ends
// multiples of 4 along the contiguous index).
template <int BX, int BR, bool RC, bool VEC>
struct TileLoad {
  static constexpr int NV = BX * BR / 4;
  static constexpr int PER = (NV + 255) / 256;
  float4 v[PER];

  __device__ __forceinline__ void load(const float* tensor, const GemmProblem&, int64_t s_x,
                                       int64_t s_r, int x0, int r0, int nx, int nr, int tid) {
    const rsrc_t rs = make_rsrc(tensor + (int64_t)x0 * s_x + (int64_t)r0 * s_r);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      int x, r;
      if (RC) { x = idx / (BR / 4); r = (idx % (BR / 4)) * 4; }
      else    { r = idx / (BX / 4); x = (idx % (BX / 4)) * 4; }
      const bool live = NV % 256 == 0 || idx < NV;
      if constexpr (VEC) {
        const bool ok = live && x < nx && r < nr;
        const uint32_t off = ok ? (uint32_t)((x * s_x + r * s_r) * 4) : kOOB;
        v[i] = bload4(rs, off);
      } else {
        float e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int xx = RC ? x : x + k, rr = RC ? r + k : r;
          const bool ok = live && xx < nx && rr < nr;
          e[k] = bload1(rs, ok ? (uint32_t)((xx * s_x + rr * s_r) * 4) : kOOB);
        }
        v[i] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }

  __device__ __forceinline__ void store(float* lds, int tid) const {
    constexpr int LD = BX + 4;   // rows stay 16-byte aligned
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      if (NV % 256 == 0 || idx < NV) {
        if (RC) {
          const int x = idx / (BR / 4), r = (idx % (BR / 4)) * 4;
          lds[(r + 0) * LD + x] = v[i].x;
          lds[(r + 1) * LD + x] = v[i].y;
          lds[(r + 2) * LD + x] = v[i].z;
          lds[(r + 3) * LD + x] = v[i].w;
        } else {
          const int r = idx / (BX / 4), x = (idx % (BX / 4)) * 4;
          *reinterpret_cast<float4*>(&lds[r * LD + x]) = v[i];
        }
      }
    }
  }
};

// Convolution operands gathered from NHWC tensors / KRSC filters.  Element
// (x, r) of the tile is tensor element (x0 + x, r0 + r) of the implicit GEMM
// operand; its offset is formed from the convolution geometry, and elements in
// the zero padding (or past the operand) read from an out-of-range offset.
// VEC: the channel count along the contiguous index is a multiple of 4, so a
// float4 never straddles two filter taps.
enum GatherKind { G_FWD_A = 1, G_DGRAD_A = 2, G_WGRAD_B = 3, G_DGRAD_B = 4 };

template <int KIND>
__device__ __forceinline__ int64_t gather_off(const GemmProblem& g, int x, int r, bool& ok) {
  // FWD_A: x = m, r = k = (tap, c).  DGRAD_A: x = m, r = k = (tap, co).
  // WGRAD_B: x = k = (tap, c), r = m.  DGRAD_B: x = c, r = k = (tap, co).
  if constexpr (KIND == G_DGRAD_B) {
    const int tap = fdiv(r, g.dCout), co = r - tap * g.cCout;
    return ((int64_t)co * 9 + tap) * g.cC + x;
  } else {
    const int m = (KIND == G_WGRAD_B) ? r : x;
    const int k = (KIND == G_WGRAD_B) ? x : r;
    const int ch = (KIND == G_DGRAD_A) ? g.cCout : g.cC;
    const FastDiv& fch = (KIND == G_DGRAD_A) ? g.dCout : g.dC;
    const int t = fdiv(m, g.dW), w = m - t * g.cW;
    const int n = fdiv(t, g.dH), h = t - n * g.cH;
    const int tap = fdiv(k, fch), c = k - tap * ch;
    const int rr = tap / 3, ss = tap - 3 * rr;
    const int hi = (KIND == G_DGRAD_A) ? h + 1 - rr : h + rr - 1;
    const int wi = (KIND == G_DGRAD_A) ? w + 1 - ss : w + ss - 1;
    ok = ok && hi >= 0 && hi < g.cH && wi >= 0 && wi < g.cW;
    return (((int64_t)n * g.cH + hi) * g.cW + wi) * ch + c;
  }
}

template <int BX, int BR, bool RC, bool VEC, int KIND>
struct GatherLoad : TileLoad<BX, BR, RC, VEC> {
  using Base = TileLoad<BX, BR, RC, VEC>;
  using Base::v;
  __device__ __forceinline__ void load(const float* tensor, const GemmProblem& g, int64_t, int64_t,
                                       int x0, int r0, int nx, int nr, int tid) {
    const rsrc_t rs = make_rsrc(tensor);
#pragma unroll
    for (int i = 0; i < Base::PER; ++i) {
      const int idx = tid + i * 256;
      int x, r;
      if (RC) { x = idx / (BR / 4); r = (idx % (BR / 4)) * 4; }
      else    { r = idx / (BX / 4); x = (idx % (BX / 4)) * 4; }
      const bool live = idx < Base::NV;
      if constexpr (VEC) {
        bool ok = live && x < nx && r < nr;
        const int64_t o = gather_off<KIND>(g, x0 + x, r0 + r, ok);
        v[i] = bload4(rs, ok ? (uint32_t)(o * 4) : kOOB);
      } else {
        float e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int xx = RC ? x : x + k, rr = RC ? r + k : r;
          bool ok = live && xx < nx && rr < nr;
          const int64_t o = gather_off<KIND>(g, x0 + xx, r0 + rr, ok);
          e[k] = bload1(rs, ok ? (uint32_t)(o * 4) : kOOB);
        }
        v[i] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
};

// Forward-fusion B operand: W tile (reduction-contiguous) with its pending
// update.  load() issues the loads of W, g, m, v; update() runs after the
// previous chunk's MFMAs, updates and writes back; store() stages the new W in LDS.
// `off` is relative to the tile's first element (row stride ldw).
template <int BX, int BR, bool VEC>
struct FFTileLoad {
  static constexpr int NV = BX * BR / 4;
  static constexpr int PER = (NV + 255) / 256;
  float4 w[PER], g[PER], m[PER], v[PER];
  int valid[PER];  // bit e set: element e of the float4 is inside the matrix
  int64_t base;    // element index of the tile origin in W

  __device__ __forceinline__ void load(const EpiArgs& ea, int64_t ldw, int x0, int r0, int nx,
                                       int nr, int tid) {
    const bool adam = ea.opt.kind != OF_OPT_SGD;
    base = (int64_t)x0 * ldw + r0;
    const rsrc_t rw = make_rsrc(ea.W.w + base), rg = make_rsrc(ea.gW + base);
    const rsrc_t rm = make_rsrc_opt(ea.W.m, base);
    const rsrc_t rv = adam ? make_rsrc(ea.W.v + base) : rm;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      const int x = idx / (BR / 4), r = (idx % (BR / 4)) * 4;
      const bool live = idx < NV && x < nx;
      if constexpr (VEC) {
        const bool ok = live && r < nr;
        valid[i] = ok ? 0xf : 0;
        const uint32_t off = ok ? (uint32_t)((x * ldw + r) * 4) : kOOB;
        w[i] = bload4(rw, off);
        g[i] = bload4(rg, off);
        m[i] = bload4(rm, off);
        v[i] = bload4(rv, off);
      } else {
        float ew[4], eg[4], em[4], ev[4];
        valid[i] = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const bool ok = live && r + k < nr;
          valid[i] |= ok ? (1 << k) : 0;
          const uint32_t off = ok ? (uint32_t)((x * ldw + r + k) * 4) : kOOB;
          ew[k] = bload1(rw, off);
          eg[k] = bload1(rg, off);
          em[k] = bload1(rm, off);
          ev[k] = bload1(rv, off);
        }
        w[i] = make_float4(ew[0], ew[1], ew[2], ew[3]);
        g[i] = make_float4(eg[0], eg[1], eg[2], eg[3]);
        m[i] = make_float4(em[0], em[1], em[2], em[3]);
        v[i] = make_float4(ev[0], ev[1], ev[2], ev[3]);
      }
    }
  }

  // Applies the update, in registers, and has its owner write it (to ea.Wout
  // when set, else in place); every workgroup feeds the updated w[] to its MFMAs.
  __device__ __forceinline__ void update(const EpiArgs& ea, int64_t ldw, int tid, bool owner) {
    const bool adam = ea.opt.kind != OF_OPT_SGD;
    const of_param& out = ea.Wout.w ? ea.Wout : ea.W;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      if (idx >= NV) continue;
      const int x = idx / (BR / 4), r = (idx % (BR / 4)) * 4;
      const int64_t o = base + (int64_t)x * ldw + r;
      float* pw = reinterpret_cast<float*>(&w[i]);
      float* pg = reinterpret_cast<float*>(&g[i]);
      float* pm = reinterpret_cast<float*>(&m[i]);
      float* pv = reinterpret_cast<float*>(&v[i]);
      if (valid[i] == 0xf && ((uintptr_t)(out.w + o) & 15u) == 0) {
        for (int e = 0; e < 4; ++e) opt_update(ea.opt, pw[e], pg[e], pm[e], pv[e]);
        if (owner) {
          st4(out.w + o, w[i]);
          if (out.m) st4(out.m + o, m[i]);
          if (adam) st4(out.v + o, v[i]);
          if (out.w_bf16) st_bf16x4(out.w_bf16 + o, w[i]);
        }
      } else if (valid[i]) {
        for (int e = 0; e < 4; ++e) {
          if (valid[i] & (1 << e)) {
            opt_update(ea.opt, pw[e], pg[e], pm[e], pv[e]);
            if (owner) {
              out.w[o + e] = pw[e];
              if (out.m) out.m[o + e] = pm[e];
              if (adam) out.v[o + e] = pv[e];
              if (out.w_bf16) out.w_bf16[o + e] = f32_to_bf16(pw[e]);
            }
          }
        }
      }
    }
  }

  // Stage the updated values in LDS as [r][x] floats (row pad 4).
  __device__ __forceinline__ void store(float* lds, int tid) const {
    constexpr int LD = BX + 4;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      if (idx >= NV) continue;
      const int x = idx / (BR / 4), r = (idx % (BR / 4)) * 4;
      lds[(r + 0) * LD + x] = w[i].x;
      lds[(r + 1) * LD + x] = w[i].y;
      lds[(r + 2) * LD + x] = w[i].z;
      lds[(r + 3) * LD + x] = w[i].w;
    }
  }
};

}  // namespace opfuse

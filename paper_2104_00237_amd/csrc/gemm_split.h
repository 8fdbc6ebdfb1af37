// fp32 contractions on the bf16 matrix cores, for products large enough that
// the matrix cores bound them.
//
// Every fp32 operand x is split into three bf16 values by truncation,
//   x = h + m + l,  h = x's top 8 significant bits, m the next 8, l the last 8,
// exactly down to 2^-110; below, bits under the smallest bf16 (2^-133) are lost.
// A product a*b is summed as eight partial products,
//   ah*bh  +  (am*bl + al*bm + al*bh + ah*bl + am*bm + am*bh + ah*bm);
// the ninth, al*bl, is below 2^-29 of it.  (Truncated parts have the operand's sign:
// leaving out am*bl and al*bm too, each below 2^-22, would make every product too
// small by up to 2^-21, eight roundings of an fp32 product.)  Products of bf16
// values are exact in fp32 and v_mfma_f32_32x32x16_bf16 accumulates in fp32; the
// leading products and the corrections have accumulators of their own, added once
// at the end, so a sum of one product is rounded once.  Eight such MFMAs cover 16
// reduction elements in 256 cycles; v_mfma_f32_32x32x2_f32 needs 512.
//
// Infinities and NaN: h of an infinite element is infinite and its m is NaN, so
// the corrections it touches become NaN, while the leading sum holds what the
// fp32 sum would; a leading sum that is not finite is therefore the result by
// itself.  h never rounds up, so the largest finite values stay finite.  A signalling
// NaN whose payload lies in the low 16 bits counts as an infinity (quieting every
// element first costs a vector instruction each, 2% to 4% of these kernels' time).
//
// What bounds it: the MFMAs (half of an fp32 MFMA's time: 314 TFLOP/s at the peak
// clock), the split (5.5 vector instructions per element) and staging between them,
// and the global loads: 168 TFLOP/s at 2048 x 4096 x 4096 (409 us; fp32 MFMA tiles
// 526, 131).  A 64x64 sub-tile per wavefront keeps LDS reads at half its bandwidth;
// two workgroups per CU fill each other's issue slots, and one alone does nearly as
// well when the split and the loads are spread between its MFMAs
// (sched_group_barrier).  A third LDS buffer with one wavefront per SIMD (operands of
// the next step read ahead) was slower by a tenth.  Errors against float64, split and
// fp32 MFMA tiles: 1024 x 2048 x 2048 forward 1.3e-7, 8.1e-7; outputs of one product
// 2.5e-8 both, of 8 products 2.8e-8, 5.4e-8.
//
// LDS: each operand tile is three planes (h, m, l) of bf16 in the operand's
// memory order.  Reduction-contiguous: rows [x][BR], whose 16-byte slots are
// XOR-swizzled so that the 16-byte reads of 16 consecutive rows cover all banks.
// Output-contiguous: rows [r][BX], their 64-byte blocks swizzled by row, read with
// the transposing ds_read_b64_tr_b16 (a 16-lane group reads a 4 x 16 block, lane i
// gets column i).
// Either way a thread's float4 becomes one 8-byte store per plane.
#pragma once

#include <algorithm>
#include <type_traits>

#include "gemm_tiles.h"

namespace opfuse {

typedef __bf16 sbf16x8_t __attribute__((ext_vector_type(8)));
typedef short sshort4_t __attribute__((ext_vector_type(4)));
typedef float sfloatx16_t __attribute__((ext_vector_type(16)));

template <int BP_, int BQ_, int BR_, int WP_, int WQ_, int WR_, int NS_, int NA_ = 1>
struct STile {
  static constexpr int BP = BP_, BQ = BQ_, BR = BR_, WP = WP_, WQ = WQ_, WR = WR_, NS = NS_;
  static constexpr int NA = NA_;   // leading sums per output element (see S64x64)
  static_assert(WP * WQ * WR == 4, "a workgroup is 4 wavefronts");
  static constexpr int WTP = BP / WP, WTQ = BQ / WQ;
  static constexpr int TP = WTP / 32, TQ = WTQ / 32;
  static_assert(TP >= 1 && TQ >= 1 && WTP % 32 == 0 && WTQ % 32 == 0, "32x32 blocks");
  static constexpr int RW = BR / WR, KS = RW / 16;   // reduction steps per wavefront and chunk
  static_assert(RW % 16 == 0 && (BR == 16 || BR == 32), "whole MFMA steps");
};

// 128x128 and 64x128: a 64x64 sub-tile per wavefront, 12 KB of LDS reads per 32
// MFMAs; in the 64-row tile two wavefronts halve each chunk's reduction and
// their sums are added in wave order.  64x64: 32x32 sub-tiles, for smaller outputs;
// its registers hold four leading sums per element (two for gradients, whose
// transposing reads need more), which take the reduction steps in turn: rounding
// errors grow with the length of a chain (1000 x 1024 x 1024 forward: 1.8e-7 with one,
// 1.0e-7 with four).
using S128x128 = STile<128, 128, 16, 2, 2, 1, 2>;
using S64x128 = STile<64, 128, 32, 1, 2, 2, 2>;
using S64x64 = STile<64, 64, 32, 2, 2, 1, 2, 4>;
// The fused forward's tiles: W, g, m and v take registers, so they are narrow.
// 128x32 stands for 128x128, 128x32N for 64x64, 128x32R and 64x32 (up to 512 rows) for
// 64x128: whole or halved chunks and leading sums as there, so every output element
// takes the same MFMA sequence as in the plain forward.  With as many columns as
// the plain tiles too few wavefronts fit (1000 x 1024 x 1024: 88 us on 64x64, 60 on
// 128x32; 512 x 4096 x 4096: 370 us with a 128x64 tile, 275; over short reductions too:
// 3322 x 264 -> 4212 261, 145, where fp32 tiles would take 129 and the plain forward gains
// as much, 92 -> 70).
using S128x32 = STile<128, 32, 32, 4, 1, 1, 2>;
using S128x32N = STile<128, 32, 32, 4, 1, 1, 2, 4>;
using S128x32R = STile<128, 32, 32, 2, 1, 2, 2>;
using S64x32 = STile<64, 32, 32, 2, 1, 2, 2>;

// A float4 as three 8-byte quads of bf16.
struct Split4 {
  uint2 h, m, l;
};

__device__ __forceinline__ uint32_t hi16(float a, float b) {   // bf16 bits of (a, b), truncated
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}

__device__ __forceinline__ float trunc16(float x) {
  return __uint_as_float(__float_as_uint(x) & 0xffff0000u);
}

__device__ __forceinline__ Split4 split4(float4 v) {
  // the two differences are exact: each only drops leading bits
  const float4 r = make_float4(__fsub_rn(v.x, trunc16(v.x)), __fsub_rn(v.y, trunc16(v.y)),
                               __fsub_rn(v.z, trunc16(v.z)), __fsub_rn(v.w, trunc16(v.w)));
  const float4 t = make_float4(__fsub_rn(r.x, trunc16(r.x)), __fsub_rn(r.y, trunc16(r.y)),
                               __fsub_rn(r.z, trunc16(r.z)), __fsub_rn(r.w, trunc16(r.w)));
  return Split4{make_uint2(hi16(v.x, v.y), hi16(v.z, v.w)), make_uint2(hi16(r.x, r.y), hi16(r.z, r.w)),
                make_uint2(hi16(t.x, t.y), hi16(t.z, t.w))};
}

// Leading sum and corrections to the result (see above for what is not finite).
__device__ __forceinline__ float split_sum(float hh, float corr) {
  return fabsf(hh) < __builtin_inff() ? __fadd_rn(hh, corr) : hh;
}

// LDS image of one operand tile: BX output rows, BR reduction elements.
template <int BX, int BR, bool RC>
struct SPlanes {
  static constexpr int ROW = RC ? BR * 2 : BX * 2;               // bytes per row
  static constexpr int PLANE = (RC ? BX : BR) * ROW;             // bytes per plane
  static constexpr int BYTES = 3 * PLANE;
  static constexpr int NV = BX * BR / 4;

  __device__ __forceinline__ static int swz(int x, int slot) {
    return slot ^ (BR == 16 ? (x >> 3) & 1 : (x >> 2) & 3);
  }

  // Output-contiguous: the 64-byte blocks of a row are XOR-swizzled so that the
  // four rows a transposing read touches lie in different banks.
  __device__ __forceinline__ static int blk(int r) {
    return (BX >= 128 ? r & 3 : BX == 64 ? (r >> 1) & 1 : 0) << 6;
  }

  // Item idx of the tile (the loaders' order) to the three planes.
  __device__ __forceinline__ static void put(char* lds, int idx, float4 v) {
    int off;
    if constexpr (RC) {
      const int x = idx / (BR / 4), r = (idx % (BR / 4)) * 4;
      off = x * ROW + swz(x, r >> 3) * 16 + (r & 4) * 2;
    } else {
      const int r = idx / (BX / 4), x = (idx % (BX / 4)) * 4;
      off = r * ROW + ((x * 2) ^ blk(r));
    }
    const Split4 s = split4(v);
    *reinterpret_cast<uint2*>(lds + off) = s.h;
    *reinterpret_cast<uint2*>(lds + off + PLANE) = s.m;
    *reinterpret_cast<uint2*>(lds + off + 2 * PLANE) = s.l;
  }

  template <int PER>
  __device__ __forceinline__ static void store(char* lds, const float4 (&v)[PER], int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + i * 256;
      if (NV % 256 == 0 || idx < NV) put(lds, idx, v[i]);
    }
  }

  // The MFMA operand of rows x0 .. x0+31 and reduction elements r0 .. r0+15 of
  // plane p: row x0 + lane%32, elements 8*(lane/32) .. +7 of the step.
  __device__ __forceinline__ static sbf16x8_t frag(const char* lds, int p, int x0, int r0, int lane) {
    const char* b = lds + p * PLANE;
    if constexpr (RC) {
      const int x = x0 + (lane & 31);
      return *reinterpret_cast<const sbf16x8_t*>(b + x * ROW + swz(x, (r0 >> 3) + (lane >> 5)) * 16);
    } else {
      const int r = r0 + (lane >> 5) * 8 + ((lane & 15) >> 2);
      const int x = x0 + (lane & 16) + (lane & 3) * 4;
      typedef __attribute__((address_space(3))) sshort4_t* lp;
      const char* a = b + r * ROW + ((x * 2) ^ blk(r));
      const sshort4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)a);
      const sshort4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a + 4 * ROW));
      typedef short sshort8_t __attribute__((ext_vector_type(8)));
      return __builtin_bit_cast(sbf16x8_t, (sshort8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

// VECS: bit 0 -- 128-bit loads of A allowed, bit 1 -- of B.
template <class T, int EPI, int VECS, bool CONV>
__global__ __launch_bounds__(256, 2) void gemm_split_kernel(GemmProblem pr, EpiArgs ea, int r_split,
                                                         float* partial, int vec_epi) {
  constexpr bool VA = (VECS & 1) != 0, VB = (VECS & 2) != 0;
  constexpr bool FF = EPI == EPI_FWD_FF;
  constexpr bool A_RC = (EPI == EPI_FWD || FF || EPI == EPI_DGRAD);
  constexpr bool B_RC = (EPI == EPI_FWD || FF);
  constexpr bool WG = (EPI == EPI_WGRAD || EPI == EPI_WGRAD_BF);
  using LA = SPlanes<T::BP, T::BR, A_RC>;
  using LB = SPlanes<T::BQ, T::BR, B_RC>;
  constexpr int STAGE = LA::BYTES + LB::BYTES;
  constexpr int LDC = T::BQ + 4;
  constexpr int PR = T::BP;
  constexpr int SM_C = T::WR * PR * LDC * 4;   // the accumulators, staged for the epilogue
  constexpr int SMX = 2 * STAGE > SM_C ? 2 * STAGE : SM_C;
  static_assert(SMX + T::BQ * 4 <= 80 * 1024, "two workgroups per CU");
  __shared__ __attribute__((aligned(16))) char smem[SMX + (FF ? T::BQ * 4 : 0)];
  float* bias_s = reinterpret_cast<float*>(smem + SMX);   // forward-fusion only
  if constexpr (EPI == EPI_FWD) {
    if ((int)blockIdx.z < ea.carry.cz) {
      carry_update(ea.carry);  // a later operator's update rides on this launch
      return;
    }
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wp = wave % T::WP, wq = (wave / T::WP) % T::WQ, wr = wave / (T::WP * T::WQ);
  int tx, ty;
  xcd_tile(tx, ty);
  const int p0 = tx * T::BP, q0 = ty * T::BQ;
  const int split = (int)blockIdx.z - ea.carry.cz, S = (int)gridDim.z - ea.carry.cz;
  const int rbeg = split * r_split;
  const int rend = min(pr.R, rbeg + r_split);
  const int nch = (rend - rbeg + T::BR - 1) / T::BR;
  const bool do_db = WG && ea.with_db && ty == 0;
  const bool ff_owner = ea.Wout.w == nullptr || p0 == 0;

  constexpr int NA = T::NA == 1 || (A_RC && B_RC) ? T::NA : 2;
  sfloatx16_t acc[NA][T::TP][T::TQ], cor[T::TP][T::TQ];
#pragma unroll
  for (int i = 0; i < T::TP; ++i)
#pragma unroll
    for (int j = 0; j < T::TQ; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        cor[i][j][k] = 0.f;
#pragma unroll
        for (int n = 0; n < NA; ++n) acc[n][i][j][k] = 0.f;
      }

  constexpr int NS = T::NS;   // chunks in the register ring
  using ALoad = std::conditional_t<
      CONV && A_RC, GatherLoad<T::BP, T::BR, true, VA, EPI == EPI_DGRAD ? G_DGRAD_A : G_FWD_A>,
      TileLoad<T::BP, T::BR, A_RC, VA>>;
  using BLoad = std::conditional_t<
      CONV && EPI == EPI_DGRAD, GatherLoad<T::BQ, T::BR, false, VB, G_DGRAD_B>,
      std::conditional_t<CONV && WG, GatherLoad<T::BQ, T::BR, false, VB, G_WGRAD_B>,
                         TileLoad<T::BQ, T::BR, B_RC, VB>>>;
  ALoad la[NS];
  BLoad lb[FF ? 1 : NS];
  FFTileLoad<T::BQ, T::BR, VB> lf[FF ? NS : 1];
  const int np = pr.P - p0, nq = pr.Q - q0;
  // column sums of dZ (the bias gradient): a thread's items all hold the same
  // four output rows
  static_assert(!WG || 256 % (T::BP / 4) == 0, "one column quad per thread");
  float dbs[4] = {0.f, 0.f, 0.f, 0.f};

  auto issue_a = [&](int slot, int c) {
    const int r0 = rbeg + c * T::BR;
    la[slot].load(pr.A, pr, pr.a_sp, pr.a_sr, p0, r0, np, c < nch ? rend - r0 : 0, tid);
  };
  auto issue_b = [&](int slot, int c) {
    const int r0 = rbeg + c * T::BR;
    const int nr = c < nch ? rend - r0 : 0;
    if constexpr (FF) lf[slot].load(ea, pr.b_sq, q0, r0, nq, nr, tid);
    else lb[slot].load(pr.B, pr, pr.b_sq, pr.b_sr, q0, r0, nq, nr, tid);
  };
  auto stage_a = [&](int slot, int c) {   // chunk c's A tile to LDS
    LA::store(smem + (c & 1) * STAGE, la[slot].v, tid);
    if constexpr (WG) {   // (without a branch on do_db, which would split the schedule)
#pragma unroll
      for (int i = 0; i < ALoad::PER; ++i) {
        dbs[0] = __fadd_rn(dbs[0], la[slot].v[i].x);
        dbs[1] = __fadd_rn(dbs[1], la[slot].v[i].y);
        dbs[2] = __fadd_rn(dbs[2], la[slot].v[i].z);
        dbs[3] = __fadd_rn(dbs[3], la[slot].v[i].w);
      }
    }
  };
  auto stage_b = [&](int slot, int c) {   // chunk c's B tile (and its update)
    char* buf = smem + (c & 1) * STAGE + LA::BYTES;
    if constexpr (FF) {
      if (c < nch) lf[slot].update(ea, pr.b_sq, tid, ff_owner);
      LB::store(buf, lf[slot].w, tid);
    } else {
      LB::store(buf, lb[slot].v, tid);
    }
  };

  // The operands of one reduction step of a wavefront.
  struct Frags {
    sbf16x8_t a[T::TP][3], b[T::TQ][3];
  };
  auto read = [&](Frags& f, int c, int k) {
    const char* a_s = smem + (c & 1) * STAGE;
    const char* b_s = a_s + LA::BYTES;
    const int r0 = wr * T::RW + k * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int i = 0; i < T::TP; ++i) f.a[i][p] = LA::frag(a_s, p, wp * T::WTP + i * 32, r0, lane);
#pragma unroll
      for (int j = 0; j < T::TQ; ++j) f.b[j][p] = LB::frag(b_s, p, wq * T::WTQ + j * 32, r0, lane);
    }
  };
  auto mm = [&](sfloatx16_t (&d)[T::TP][T::TQ], const Frags& f, int pa, int pb) {
#pragma unroll
    for (int i = 0; i < T::TP; ++i)
#pragma unroll
      for (int j = 0; j < T::TQ; ++j)
        d[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i][pa], f.b[j][pb], d[i][j], 0, 0, 0);
  };

#pragma unroll
  for (int s = 0; s < NS; ++s) {
    issue_a(s, s);
    issue_b(s, s);
    __builtin_amdgcn_sched_barrier(0);   // chunk 0 stays the oldest load
  }
  if (FF || EPI == EPI_WGRAD_BF) opt_prepare(ea.opt);
  stage_a(0, 0);
  stage_b(0, 0);
  __syncthreads();

  // Chunk c from slot s (s == c % NS, a constant): its operands are read from
  // LDS, chunk c+NS is requested, and chunk c+1 is split and stored to the other
  // buffer between the MFMAs.  One barrier per chunk.
  auto chunk = [&](const int c, const int s) {
    Frags f[T::KS];
    constexpr int RA = A_RC ? 1 : 2, RB = B_RC ? 1 : 2;          // LDS reads per operand
    constexpr int NM = 8 * T::KS * T::TP * T::TQ;                // MFMAs per chunk
    constexpr int R0 = T::TP * RA + T::TQ * RB, NRD = 3 * T::KS * R0;
#pragma unroll
    for (int k = 0; k < T::KS; ++k) read(f[k], c, k);
    issue_a(s, c + NS);   // slot s held chunk c, already in LDS
    issue_b(s, c + NS);
    stage_a((s + 1) % NS, c + 1);
    stage_b((s + 1) % NS, c + 1);
#pragma unroll
    for (int k = 0; k < T::KS; ++k) {
      mm(acc[(s * T::KS + k) % NA], f[k], 0, 0);
      mm(cor, f[k], 2, 1);
      mm(cor, f[k], 1, 2);
      mm(cor, f[k], 2, 0);
      mm(cor, f[k], 0, 2);
      mm(cor, f[k], 1, 1);
      mm(cor, f[k], 1, 0);
      mm(cor, f[k], 0, 1);
    }
    if constexpr (!FF) {
      // after the first operands: one MFMA, then its share of the LDS reads, of
      // the loads, of the split's vector instructions and of the LDS stores
      constexpr int NEL = (T::BP + T::BQ) * T::BR / 1024;         // float4s split per chunk
      // (26 vector instructions split and pack a float4; four single loads in its
      // place need 16 more for their addresses)
      constexpr int NV = (NEL * (VECS == 3 ? 26 : 42) + NM - 1) / NM;
      __builtin_amdgcn_sched_group_barrier(0x100, R0, 0);
#pragma unroll
      for (int g = 0; g < NM; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, (NRD - R0) * 3 / NM + 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);
        if (g > 3) __builtin_amdgcn_sched_group_barrier(0x200, (NEL * 3 + NM - 5) / (NM - 4), 0);
      }
    }
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };
  const int nfull = nch / NS * NS;
  for (int c0 = 0; c0 < nfull; c0 += NS) {
#pragma unroll
    for (int s = 0; s < NS; ++s) chunk(c0 + s, s);
  }
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (nfull + s < nch) chunk(nfull + s, s);

  // Epilogue: the results go through LDS in row-major order, whole tile
  // (MFMA 32x32 layout: lane holds column lane%32, rows 8*(k/4) + 4*(lane/32) + k%4).
  float* Cs = reinterpret_cast<float*>(smem);
  constexpr int NQ4 = T::BQ / 4;
  constexpr int ITEMS = PR * NQ4;
  constexpr int EPT = (ITEMS + 255) / 256;

  const bool ff_bias = FF && ea.b.w != nullptr;
  if (ff_bias && split == 0 && tid < T::BQ && q0 + tid < pr.Q) {
    const int i = q0 + tid;
    const bool adam = ea.opt.kind != OF_OPT_SGD;
    float w = ea.b.w[i], m = ea.b.m ? ea.b.m[i] : 0.f, v = adam ? ea.b.v[i] : 0.f;
    opt_update(ea.opt, w, ea.gb[i], m, v);
    if (ff_owner) {
      const of_param& out = ea.bout.w ? ea.bout : ea.b;
      out.w[i] = w;
      if (out.m) out.m[i] = m;
      if (adam) out.v[i] = v;
      if (out.w_bf16) out.w_bf16[i] = f32_to_bf16(w);
    }
    bias_s[tid] = w;
  }

  {
#pragma unroll
    for (int i = 0; i < T::TP; ++i)
#pragma unroll
      for (int j = 0; j < T::TQ; ++j)
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int p = wp * T::WTP + i * 32 + (k >> 2) * 8 + (lane >> 5) * 4 + (k & 3);
          const int q = wq * T::WTQ + j * 32 + (lane & 31);
          float hh = acc[0][i][j][k];
#pragma unroll
          for (int n = 1; n < NA; ++n) hh = __fadd_rn(hh, acc[n][i][j][k]);
          Cs[(wr * PR + p) * LDC + q] = split_sum(hh, cor[i][j][k]);
        }
    __syncthreads();
    auto item = [&](int idx, float (&c)[4]) {   // results of item idx of the band
      const int p = idx / NQ4, q = (idx % NQ4) * 4;
      float4 s = *reinterpret_cast<const float4*>(&Cs[p * LDC + q]);
#pragma unroll
      for (int w2 = 1; w2 < T::WR; ++w2) {
        const float4 t = *reinterpret_cast<const float4*>(&Cs[(w2 * PR + p) * LDC + q]);
        s.x = __fadd_rn(s.x, t.x); s.y = __fadd_rn(s.y, t.y);
        s.z = __fadd_rn(s.z, t.z); s.w = __fadd_rn(s.w, t.w);
      }
      c[0] = s.x; c[1] = s.y; c[2] = s.z; c[3] = s.w;
    };
    // A group of items' operands (parameter and history, or the saved tensor)
    // are requested together, then used: item by item, each item's loads
    // would wait behind the previous item's stores.
    constexpr int G = EPT < 8 ? EPT : 8;
    const bool grp_bf = EPI == EPI_WGRAD_BF && S == 1 && (vec_epi & 2) && (pr.Q & 3) == 0;
    const bool grp_dg = EPI == EPI_DGRAD && S == 1 && (vec_epi & 1) && (pr.Q & 3) == 0 &&
                        ea.act != OF_ACT_NONE && ea.res == nullptr;
    if (grp_bf || grp_dg) {
      if constexpr (EPI == EPI_WGRAD_BF || EPI == EPI_DGRAD) {
        constexpr bool BF = EPI == EPI_WGRAD_BF;
        const int64_t ld = BF ? ea.ldo : ea.ldp;
        const int64_t org = (int64_t)p0 * ld + q0;
        const rsrc_t rw = make_rsrc(BF ? ea.W.w + org : ea.prev + org);
        const rsrc_t rm = BF ? make_rsrc_opt(ea.W.m, org) : rw;
        const rsrc_t rv = BF && ea.opt.kind != OF_OPT_SGD ? make_rsrc(ea.W.v + org) : rm;
        const rsrc_t rg = BF ? make_rsrc_opt(ea.gW, org) : rm;   // no earlier use: reads 0
#pragma unroll
        for (int e0 = 0; e0 < EPT; e0 += G) {
          float4 pw[G], pm[G], pv[G], pg[G];
#pragma unroll
          for (int u = 0; u < G; ++u) {
            const int idx = tid + (e0 + u) * 256;
            const int p = idx / NQ4, q = (idx % NQ4) * 4;
            const bool ok = e0 + u < EPT && idx < ITEMS && p0 + p < pr.P && q0 + q < pr.Q;
            const uint32_t off = ok ? (uint32_t)((p * ld + q) * 4) : kOOB;
            pw[u] = bload4(rw, off);
            if constexpr (BF) {
              pm[u] = bload4(rm, off);
              pv[u] = bload4(rv, off);
              pg[u] = bload4(rg, off);
            }
          }
#pragma unroll
          for (int u = 0; u < G; ++u) {
            const int idx = tid + (e0 + u) * 256;
            if (e0 + u >= EPT || idx >= ITEMS) break;
            const int gp = p0 + idx / NQ4, gq = q0 + (idx % NQ4) * 4;
            if (gp >= pr.P || gq >= pr.Q) continue;
            float c[4];
            item(idx, c);
            const int64_t oo = (int64_t)gp * ea.ldo + gq;
            if constexpr (BF) {
              if (ea.gW) {
                c[0] = __fadd_rn(pg[u].x, c[0]); c[1] = __fadd_rn(pg[u].y, c[1]);
                c[2] = __fadd_rn(pg[u].z, c[2]); c[3] = __fadd_rn(pg[u].w, c[3]);
              }
              opt_apply4(ea.opt, ea.W, OptState4{pw[u], pm[u], pv[u]},
                         make_float4(c[0], c[1], c[2], c[3]), oo);
            } else {
              st4(ea.out + oo, make_float4(__fmul_rn(c[0], act_grad(ea.act, pw[u].x)),
                                           __fmul_rn(c[1], act_grad(ea.act, pw[u].y)),
                                           __fmul_rn(c[2], act_grad(ea.act, pw[u].z)),
                                           __fmul_rn(c[3], act_grad(ea.act, pw[u].w))));
            }
          }
        }
      }
    } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int idx = tid + e * 256;
      if (ITEMS % 256 != 0 && idx >= ITEMS) break;
      const int q = (idx % NQ4) * 4;
      const int gp = p0 + idx / NQ4, gq = q0 + q;
      if (gp >= pr.P || gq >= pr.Q) continue;
      float c[4];
      item(idx, c);
      const int n = min(4, pr.Q - gq);
      if (S > 1) {
        float* dst = partial + ((int64_t)split * pr.P + gp) * pr.Q + gq;
        if (n == 4 && (pr.Q & 3) == 0) st4(dst, make_float4(c[0], c[1], c[2], c[3]));
        else for (int k = 0; k < n; ++k) dst[k] = c[k];
      } else {
        const float* bias = nullptr;
        if (EPI == EPI_FWD && ea.bias) bias = ea.bias + gq;
        if (ff_bias) bias = bias_s + q;
        epilogue<EPI>(ea, gp, gq, c, n, bias, vec_epi);
      }
    }
    }
  }

  if (do_db) {
    // Bias gradient: the threads' column sums, added in thread order.
    __syncthreads();
    constexpr int NG = 1024 / T::BP;   // threads per column quad
    float* red = reinterpret_cast<float*>(smem);   // [NG][BP]
    const int x = (tid % (T::BP / 4)) * 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) red[(tid / (T::BP / 4)) * T::BP + x + k] = dbs[k];
    __syncthreads();
    if (tid < T::BP && p0 + tid < pr.P) {
      float s = red[tid];
#pragma unroll
      for (int g = 1; g < NG; ++g) s = __fadd_rn(s, red[g * T::BP + tid]);
      if (S > 1) partial[(int64_t)S * pr.P * pr.Q + (int64_t)split * pr.P + p0 + tid] = s;
      else bias_epilogue<EPI>(ea, p0 + tid, s);
    }
  }
}

template <class T, int EPI, bool CONV>
static hipError_t split_launch_t(int S, int cz, int r_split, const GemmProblem& pr, const EpiArgs& ea,
                                 void* ws, int vec_ops, int vec_epi, hipStream_t s) {
  const dim3 grid((pr.P + T::BP - 1) / T::BP, (pr.Q + T::BQ - 1) / T::BQ, S + cz);
  if (vec_ops == 3) {
    hipLaunchKernelGGL((gemm_split_kernel<T, EPI, 3, CONV>), grid, dim3(256), 0, s, pr, ea, r_split,
                       (float*)ws, vec_epi);
  } else if (CONV && vec_ops == 1) {
    // a convolution's two channel counts can differ in their alignment
    if constexpr (CONV)
      hipLaunchKernelGGL((gemm_split_kernel<T, EPI, 1, CONV>), grid, dim3(256), 0, s, pr, ea, r_split,
                         (float*)ws, vec_epi);
  } else if (CONV && vec_ops == 2) {
    if constexpr (CONV)
      hipLaunchKernelGGL((gemm_split_kernel<T, EPI, 2, CONV>), grid, dim3(256), 0, s, pr, ea, r_split,
                         (float*)ws, vec_epi);
  } else {
    hipLaunchKernelGGL((gemm_split_kernel<T, EPI, 0, CONV>), grid, dim3(256), 0, s, pr, ea, r_split,
                       (float*)ws, vec_epi);
  }
  return hipGetLastError();
}

// One contraction; the tiles each kind takes: see cheapest_split and gemm_launch.
enum SplitTile { ST_128x128 = 0, ST_64x128, ST_64x64, ST_64x32, ST_128x32, ST_128x32N, ST_128x32R, ST_COUNT };

template <int EPI, bool CONV>
static hipError_t split_launch_kind(int tile, int S, int cz, int r_split, const GemmProblem& pr,
                                    const EpiArgs& ea, void* ws, int vo, int ve, hipStream_t s) {
  if constexpr (EPI == EPI_FWD_FF) {
    if (tile == ST_64x32) return split_launch_t<S64x32, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32) return split_launch_t<S128x32, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32N) return split_launch_t<S128x32N, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x32R) return split_launch_t<S128x32R, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  } else {
    if (tile == ST_64x64) return split_launch_t<S64x64, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
    if (tile == ST_128x128) return split_launch_t<S128x128, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  if constexpr (EPI == EPI_FWD || EPI == EPI_DGRAD) {
    if (tile == ST_64x128) return split_launch_t<S64x128, EPI, CONV>(S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  return hipErrorInvalidValue;
}

template <bool CONV>
static hipError_t split_launch(int kind, int tile, int S, int cz, int r_split, const GemmProblem& pr,
                               const EpiArgs& ea, void* ws, int vo, int ve, hipStream_t s) {
  switch (kind) {
    case EPI_FWD: return split_launch_kind<EPI_FWD, CONV>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_FWD_FF: return split_launch_kind<EPI_FWD_FF, CONV>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_DGRAD: return split_launch_kind<EPI_DGRAD, CONV>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_WGRAD: return split_launch_kind<EPI_WGRAD, CONV>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
    case EPI_WGRAD_BF: return split_launch_kind<EPI_WGRAD_BF, CONV>(tile, S, cz, r_split, pr, ea, ws, vo, ve, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace opfuse

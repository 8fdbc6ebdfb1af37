// bf16-operand forward and data gradient on 256x256 tiles (v_mfma_f32_32x32x16_bf16).
//
// What bounds these products on smaller tiles is a CU's load-return path (64 B per
// clock): a 128x128 tile asks it for as many cycles as its MFMAs take, a 256x256
// tile for half.  Four wavefronts, one per SIMD, each hold a 128x128 sub-tile
// (256 accumulator registers); 16 MFMAs take 8 KB of LDS reads, half of LDS's rate.
//
// bf16 operands go from memory straight to LDS (16 bytes a lane, no registers);
// an fp32 operand (dZ, or X stored as fp32) goes through registers, rounded to
// nearest even on the way, as in the general kernel.  LDS holds two chunks of 64
// reduction elements.  One barrier per chunk, before its last step:
//   step 0..2 of chunk c   MFMAs of step k, LDS reads of step k+1
//   barrier                chunk c+1 has landed, chunk c has been read
//   step 3                 MFMAs, reads of chunk c+1's step 0; chunk c+2 is requested
// so a chunk has the time of a whole chunk to arrive (fp32: rounded and stored
// during steps 0..2 of the chunk after its loads were issued).  The two buffers are
// arrays of their own: the compiler then knows which reads a load to LDS concerns.
//
// Measured: 4096 x 4096 x 1024 forward with GELU, Z and a bf16 Y 75 -> 58 us (100 MB of
// stores; the MFMAs are a fifth of it); a data gradient of that size with GELU's
// derivative 93 -> 55.  Below 160 tiles the chip is not full and the general kernel's
// smaller tiles win.  A long forward is split as there (4096 x 4096 x 8192 395 -> 360 us).
//
// LDS layout: reduction-contiguous operands as rows [x][64], 16-byte slots
// XOR-swizzled by (x >> 1) & 7, so 16 consecutive rows' reads cover all banks;
// output-contiguous ones (the data gradient's W) as rows [r][256], 64-byte blocks
// swizzled by r & 3, read with ds_read_b64_tr_b16.  A load to LDS writes lane i at
// base + 16 i, so the swizzle is applied to the address each lane loads from.

#include <type_traits>
#include <utility>

#include "gemm_common.h"

namespace opfuse {

typedef __bf16 wbf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 wbf16x2_t __attribute__((ext_vector_type(2)));
typedef float wfloat2_t __attribute__((ext_vector_type(2)));
typedef short wshort4_t __attribute__((ext_vector_type(4)));
typedef short wshort8_t __attribute__((ext_vector_type(8)));
typedef float wfloatx16_t __attribute__((ext_vector_type(16)));

namespace {

constexpr int BT = 256;                 // tile rows and columns
constexpr int BR = 64;                  // reduction elements per chunk
constexpr int OPB = BT * BR * 2;        // bytes of one operand's chunk in LDS

__device__ __forceinline__ uint32_t cvt2(float a, float b) {   // round to nearest even
  const wfloat2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, wbf16x2_t));
}

// Direct loads of one operand's chunks to LDS: 32 KB, 8 instructions of 1 KB per
// wavefront.  A lane's offsets from the chunk are the same for every chunk.
// ld: row stride in elements; nx: rows (RC) or columns inside the operand.
template <bool RC>
struct Dma {
  uint32_t off[8];
  int r[8];

  __device__ __forceinline__ Dma(int64_t ld, int nx, int lane, int wave) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int blk = wave * 8 + i;       // 1 KB block of the chunk
      int x;
      if constexpr (RC) {
        x = blk * 8 + (lane >> 3);
        r[i] = (((lane & 7) ^ ((x >> 1) & 7)) * 8);
        off[i] = x < nx ? (uint32_t)((x * ld + r[i]) * 2) : kOOB;
      } else {
        r[i] = blk * 2 + (lane >> 5);
        x = (((lane & 31) >> 2) ^ (r[i] & 3)) * 32 + (lane & 3) * 8;
        off[i] = x < nx ? (uint32_t)((r[i] * ld + x) * 2) : kOOB;
      }
    }
  }
  // nr: reduction elements of the chunk inside the operand; soff: the chunk's offset.
  __device__ __forceinline__ void operator()(char* lds, const rsrc_t& rs, int nr, uint32_t soff,
                                             int wave) const {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(lds + (wave * 8 + i) * 1024), 16,
          r[i] < nr ? off[i] : kOOB, soff, 0, 0);
  }
};

// fp32 chunk (reduction-contiguous) through registers: 16 float4s per thread.
struct Reg32 {
  float4 v[16];
  __device__ __forceinline__ void load(const rsrc_t& rs, int64_t ld, int r0, int nx, int nr, int tid) {
    const int r = (tid & 15) * 4;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int x = (tid >> 4) + i * 16;
      v[i] = bload4(rs, x < nx && r < nr ? (uint32_t)((x * ld + r0 + r) * 4) : kOOB);
    }
  }
  template <int I0, int I1>
  __device__ __forceinline__ void store(char* lds, int tid) const {
    const int r = (tid & 15) * 4;
#pragma unroll
    for (int i = I0; i < I1; ++i) {
      const int x = (tid >> 4) + i * 16;
      *reinterpret_cast<uint2*>(lds + x * 128 + ((r >> 3) ^ ((x >> 1) & 7)) * 16 + (r & 4) * 2) =
          make_uint2(cvt2(v[i].x, v[i].y), cvt2(v[i].z, v[i].w));
    }
  }
};

// f(0), f(1), ... with constants: accumulators are indexed statically.
template <int... T, class F>
__device__ __forceinline__ void each(std::integer_sequence<int, T...>, F&& f) {
  (f(std::integral_constant<int, T>{}), ...);
}

template <bool RC>
__device__ __forceinline__ wbf16x8_t frag(const char* lds, int x0, int k, int lane) {
  if constexpr (RC) {
    const int x = x0 + (lane & 31);
    return *reinterpret_cast<const wbf16x8_t*>(lds + x * 128 + ((2 * k + (lane >> 5)) ^ ((x >> 1) & 7)) * 16);
  } else {
    const int r = k * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    const int x = x0 + (lane & 16) + (lane & 3) * 4;
    const char* a = lds + r * 512 + ((x * 2) ^ ((r & 3) << 6));
    typedef __attribute__((address_space(3))) wshort4_t* lp;
    const wshort4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)a);
    const wshort4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a + 4 * 512));
    return __builtin_bit_cast(wbf16x8_t, (wshort8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

}  // namespace

// EPI_FWD (A = X, B = W, both reduction-contiguous) or EPI_DGRAD (A = dZ, B = W
// output-contiguous).  A32: A is stored as fp32.  ACT: a data gradient's
// activation derivative (its saved tensor's loads); RES: a residual is added.  A split
// forward's workgroups store their sums one after the other in ea.out (dense).
template <int EPI, bool A32, int ACT, bool RES>
__global__ __launch_bounds__(256, 1) void gemm_bf16_wide_kernel(GemmProblem pr, EpiArgs ea, int r_split) {
  constexpr bool B_RC = EPI == EPI_FWD;
  __shared__ __attribute__((aligned(1024))) char sa0[OPB], sa1[OPB], sb0[OPB], sb1[OPB];
  if constexpr (EPI == EPI_FWD) {
    if ((int)blockIdx.z < ea.carry.cz) {
      carry_update(ea.carry);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave & 1, wq = wave >> 1;
  int tx, ty;
  xcd_tile(tx, ty);
  const int p0 = tx * BT, q0 = ty * BT;
  const int np = pr.P - p0, nq = pr.Q - q0;
  if constexpr (EPI == EPI_FWD) {   // this split's part of the reduction
    const int split = (int)blockIdx.z - ea.carry.cz, rbeg = split * r_split;
    pr.A = (const float*)((const char*)pr.A + (int64_t)rbeg * (A32 ? 4 : 2));
    pr.B = (const float*)((const char*)pr.B + (int64_t)rbeg * 2);
    pr.R = min(r_split, pr.R - rbeg);
    ea.out += (int64_t)split * pr.P * pr.Q;
  }
  const int nch = (pr.R + BR - 1) / BR;
  const int64_t lda = pr.a_sp, ldb = B_RC ? pr.b_sq : pr.b_sr;
  const rsrc_t ra = make_rsrc((const char*)pr.A + (int64_t)p0 * lda * (A32 ? 4 : 2));
  const rsrc_t rb = make_rsrc((const char*)pr.B + (int64_t)q0 * (B_RC ? ldb : 1) * 2);

  const Dma<true> da(lda, np, lane, wave);       // unused when A is fp32
  const Dma<B_RC> db(ldb, nq, lane, wave);
  Reg32 reg[1];

  wfloatx16_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.f;
  struct Frags {
    wbf16x8_t a[4], b[4];
  };
  Frags f[2];

  auto nr_of = [&](int c) { return c < nch ? min(BR, pr.R - c * BR) : 0; };
  auto request = [&](char* a, char* b, int c) {    // chunk c to LDS (A as fp32: not here)
    const int nr = nr_of(c);   // 0 past the end: zeros
    if constexpr (!A32) da(a, ra, nr, (uint32_t)c * (BR * 2), wave);
    db(b, rb, nr, nr == 0 ? 0u : B_RC ? (uint32_t)c * (BR * 2) : (uint32_t)(c * BR * ldb * 2), wave);
  };
  auto read = [&](Frags& d, const char* a, const char* b, int k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) d.a[i] = frag<true>(a, wp * 128 + i * 32, k, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) d.b[j] = frag<B_RC>(b, wq * 128 + j * 32, k, lane);
  };
  auto mfma = [&](const Frags& d) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d.a[i], d.b[j], acc[i][j], 0, 0, 0);
  };
  auto sync = [&]() {   // this wavefront's loads to LDS and LDS accesses done, then everyone's
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(A32 ? 16 : 0) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // one MFMA, then its share of the LDS reads, of the rounding, of the LDS stores
  auto sched = [&](bool fill, bool loads) {
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (loads) {
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      if (A32 && fill) {
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // Chunk c is in (a, b); chunk c+1 lands in (an, bn).
  auto chunk = [&](char* a, char* b, char* an, char* bn, int c) {
    read(f[1], a, b, 1);
    if constexpr (A32) reg[0].template store<0, 6>(an, tid);
    mfma(f[0]);
    sched(true, false);
    read(f[0], a, b, 2);
    if constexpr (A32) reg[0].template store<6, 11>(an, tid);
    mfma(f[1]);
    sched(true, false);
    read(f[1], a, b, 3);
    if constexpr (A32) {
      reg[0].template store<11, 16>(an, tid);
      reg[0].load(ra, lda, (c + 2) * BR, np, nr_of(c + 2), tid);
    }
    mfma(f[0]);
    sched(true, false);
    sync();
    request(a, b, c + 2);
    read(f[0], an, bn, 0);
    mfma(f[1]);
    sched(false, true);
  };

  if constexpr (A32) {
    reg[0].load(ra, lda, 0, np, nr_of(0), tid);
    request(sa0, sb0, 0);
    reg[0].template store<0, 16>(sa0, tid);
    request(sa1, sb1, 1);
    reg[0].load(ra, lda, BR, np, nr_of(1), tid);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  } else {
    request(sa0, sb0, 0);
    request(sa1, sb1, 1);
    asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  __builtin_amdgcn_sched_barrier(0);
  read(f[0], sa0, sb0, 0);
  __builtin_amdgcn_sched_barrier(0);
  // (a chunk past the end is zeros: a branch around it makes the compiler move
  // accumulators between register files)
  for (int c = 0; c < nch; c += 2) {
    chunk(sa0, sb0, sa1, sb1, c);
    chunk(sa1, sb1, sa0, sb0, c + 1);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // Epilogue straight from the accumulators (lane: column lane%32, rows
  // 8*(k/4) + 4*(lane/32) + k%4 of a 32x32 block): one wavefront per SIMD has nothing
  // to hide barriers and LDS round trips behind.  A store instruction covers two
  // whole 128-byte row segments.  The saved tensor and the residual are requested
  // D - 1 blocks ahead.  Rows past P lie beyond the
  // descriptors, columns past Q get an offset beyond them.
  const int c32 = lane & 31, r4 = (lane >> 5) * 4;
  const int prow = p0 + wp * 128, qcol = q0 + wq * 128;
  const int nrow = min(128, pr.P - prow), ncol = min(128, pr.Q - qcol);   // of this sub-tile
  if (nrow <= 0 || ncol <= 0) return;
  auto desc = [&](const void* t, int64_t ld, int es) {
    return make_rsrc((const char*)t + ((int64_t)prow * ld + qcol) * es,
                     (int)(((int64_t)(nrow - 1) * ld + ncol) * es));
  };
  constexpr bool dact = EPI == EPI_DGRAD && ACT != OF_ACT_NONE, res = RES;
  const rsrc_t ro = EPI == EPI_FWD && ea.yb ? desc(ea.yb, ea.ldo, 2) : desc(ea.out, ea.ldo, 4);
  const rsrc_t rz = EPI == EPI_FWD && ea.z ? desc(ea.z, ea.ldz, 4) : ro;
  const rsrc_t rp = dact ? desc(ea.prev, ea.ldp, 4) : ro;
  const rsrc_t rr = res ? desc(ea.res, ea.ldr, 4) : ro;
  auto loc = [&](int64_t ld, int j, int es) -> uint32_t {   // this lane's first element of column block j
    return j * 32 + c32 < ncol ? (uint32_t)((r4 * ld + j * 32 + c32) * es) : kOOB;
  };
  // offset of register k of row block i (all in the vector offset, which the
  // descriptor's end is checked against; a row past P is beyond it)
  auto row = [&](int64_t ld, int i, int k, int es) -> uint32_t {
    return (uint32_t)((i * 32 + (k >> 2) * 8 + (k & 3)) * ld * es);
  };
  constexpr int D = dact && res ? 2 : 4;   // blocks in flight (4 KB each per wavefront)
  float sv[D][16], rs[D][16];
  auto fetch = [&](int t) {   // block t = 4 i + j
    const int i = t >> 2, j = t & 3;
    if constexpr (dact) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        sv[t % D][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                           rp, loc(ea.ldp, j, 4) + row(ea.ldp, i, k, 4), 0, 0));
    }
    if constexpr (res) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        rs[t % D][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                           rr, loc(ea.ldr, j, 4) + row(ea.ldr, i, k, 4), 0, 0));
    }
  };
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
  if (EPI == EPI_FWD && ea.bias) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j * 32 + c32 < ncol) bias[j] = ea.bias[qcol + j * 32 + c32];
  }
  // bf16 Y: lanes 2l and 2l+1 trade a value so that each stores two columns of a row
  const bool pair = EPI == EPI_FWD && ea.yb && ea.ldo % 2 == 0 && ((uintptr_t)ea.yb & 3u) == 0 &&
                    (ncol & 1) == 0;
#pragma unroll
  for (int t = 0; t < D - 1; ++t) fetch(t);
  auto block = [&](auto T_) {
    constexpr int t = decltype(T_)::value, i = t >> 2, j = t & 3;
    if constexpr (t + D - 1 < 16) fetch(t + D - 1);
    float c[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      c[k] = acc[i][j][k];
      if constexpr (EPI == EPI_FWD) {
        if (ea.bias) c[k] = __fadd_rn(c[k], bias[j]);
        if (ea.z)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c[k]), rz,
                                                loc(ea.ldz, j, 4) + row(ea.ldz, i, k, 4), 0, 2);
      }
    }
    if constexpr (EPI == EPI_FWD) {
      if (ea.act == OF_ACT_GELU) {
#pragma unroll
        for (int k = 0; k < 16; ++k) c[k] = act_fwd(OF_ACT_GELU, c[k]);
      } else if (ea.act == OF_ACT_RELU) {
#pragma unroll
        for (int k = 0; k < 16; ++k) c[k] = act_fwd(OF_ACT_RELU, c[k]);
      }
    } else if constexpr (dact) {
#pragma unroll
      for (int k = 0; k < 16; ++k) c[k] = __fmul_rn(c[k], act_grad(ACT, sv[t % D][k]));
    }
    if constexpr (res) {
#pragma unroll
      for (int k = 0; k < 16; ++k) c[k] = __fadd_rn(c[k], rs[t % D][k]);
    }
    if (EPI == EPI_FWD && ea.yb) {
      const uint32_t off = loc(ea.ldo, j, 2);
      if (pair) {
        const bool odd = lane & 1;
        const uint32_t poff = off == kOOB ? kOOB : off + (odd ? (uint32_t)(ea.ldo * 2) - 2u : 0u);
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          const float mine = odd ? c[k + 1] : c[k], give = odd ? c[k] : c[k + 1];
          const float got = __int_as_float(
              __builtin_amdgcn_mov_dpp(__float_as_int(give), 0xb1, 0xf, 0xf, true));   // lane ^ 1
          __builtin_amdgcn_raw_buffer_store_b32(odd ? cvt2(got, mine) : cvt2(mine, got), ro,
                                                poff + row(ea.ldo, i, k, 2), 0, 0);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 16; ++k)
          __builtin_amdgcn_raw_buffer_store_b16((short)(cvt2(c[k], 0.f) & 0xffffu), ro,
                                                off + row(ea.ldo, i, k, 2), 0, 0);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c[k]), ro,
                                              loc(ea.ldo, j, 4) + row(ea.ldo, i, k, 4), 0, 2);
    }
  };
  each(std::make_integer_sequence<int, 16>{}, block);
}

// ------------------------------------------------------------ weight gradient
// dW[p, q] = sum_r dZ[r, p] X[r, q] on 128x128 tiles, both operands output-
// contiguous: dZ (fp32) through registers, X (bf16) straight to LDS, both read with
// ds_read_b64_tr_b16; the main loop is the one above with 64x64 sub-tiles.  The
// update runs on the accumulators: W, m and v are requested a 32x32 block ahead
// and moved in 128-byte row segments.  Bound by LDS and the loads (by count 768 clocks
// of either per chunk, 512 of MFMAs), then by the update's memory traffic: 1024 x 4096
// over 4096 rows with AdamW 95 -> 78 us, the plain gradient 80 -> 55.
namespace {

constexpr int WT = 128;                  // tile rows and columns
constexpr int WOPB = WT * BR * 2;        // bytes of one operand's chunk in LDS

__device__ __forceinline__ wbf16x8_t wfrag(const char* lds, int x0, int k, int lane) {
  const int r = k * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
  const int x = x0 + (lane & 16) + (lane & 3) * 4;
  const char* a = lds + r * 256 + ((x * 2) ^ ((r & 3) << 6));
  typedef __attribute__((address_space(3))) wshort4_t* lp;
  const wshort4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)a);
  const wshort4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a + 4 * 256));
  return __builtin_bit_cast(wbf16x8_t, (wshort8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace

template <int EPI>
__global__ __launch_bounds__(256, 1) void wgrad_bf16_kernel(GemmProblem pr, EpiArgs ea) {
  static_assert(EPI == EPI_WGRAD || EPI == EPI_WGRAD_BF, "weight gradients");
  constexpr bool BF = EPI == EPI_WGRAD_BF;
  __shared__ __attribute__((aligned(1024))) char sa0[WOPB], sa1[WOPB], sb0[WOPB], sb1[WOPB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave & 1, wq = wave >> 1;
  int tx, ty;
  xcd_tile(tx, ty);
  const int p0 = tx * WT, q0 = ty * WT;
  const int np = pr.P - p0, nq = pr.Q - q0;
  const int nch = (pr.R + BR - 1) / BR;
  const rsrc_t ra = make_rsrc(pr.A + p0);
  const rsrc_t rb = make_rsrc((const char*)pr.B + (int64_t)q0 * 2);
  const int64_t lda = pr.a_sr, ldb = pr.b_sr;

  float4 reg[8];
  float dbs[4] = {0.f, 0.f, 0.f, 0.f};   // column sums of dZ: a thread's quads share their columns
  const int ax = (tid & 31) * 4, ar = tid >> 5;
  auto row_of = [&](int i) { return (i >> 2) * 32 + ar * 4 + (i & 3); };   // quad i's row of the chunk
  auto nr_of = [&](int c) { return c < nch ? min(BR, pr.R - c * BR) : 0; };
  auto load = [&](int c) {
    const int nr = nr_of(c);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = row_of(i);
      reg[i] = bload4(ra, ax < np && r < nr ? (uint32_t)((((int64_t)c * BR + r) * lda + ax) * 4) : kOOB);
    }
  };
  auto put = [&](char* lds, int i) {   // quad i, rounded to nearest even
    const int r = row_of(i);
    *reinterpret_cast<uint2*>(lds + r * 256 + ((ax * 2) ^ ((r & 3) << 6))) =
        make_uint2(cvt2(reg[i].x, reg[i].y), cvt2(reg[i].z, reg[i].w));
    if ((i & 3) == 3) {   // four rows at a time: the order of the general kernel's sums
      const float4 &s0 = reg[i - 3], &s1 = reg[i - 2], &s2 = reg[i - 1], &s3 = reg[i];
      dbs[0] = __fadd_rn(dbs[0], __fadd_rn(__fadd_rn(__fadd_rn(s0.x, s1.x), s2.x), s3.x));
      dbs[1] = __fadd_rn(dbs[1], __fadd_rn(__fadd_rn(__fadd_rn(s0.y, s1.y), s2.y), s3.y));
      dbs[2] = __fadd_rn(dbs[2], __fadd_rn(__fadd_rn(__fadd_rn(s0.z, s1.z), s2.z), s3.z));
      dbs[3] = __fadd_rn(dbs[3], __fadd_rn(__fadd_rn(__fadd_rn(s0.w, s1.w), s2.w), s3.w));
    }
  };
  uint32_t boff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 4 + (lane >> 4);
    const int x = (((lane & 15) >> 2) ^ (r & 3)) * 32 + (lane & 3) * 8;
    boff[i] = x < nq ? (uint32_t)((r * ldb + x) * 2) : kOOB;
  }
  auto request = [&](char* b, int c) {
    const int nr = nr_of(c);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rb, (__attribute__((address_space(3))) void*)(b + (wave * 4 + i) * 1024), 16,
          (wave * 4 + i) * 4 + (lane >> 4) < nr ? boff[i] : kOOB, nr ? (uint32_t)(c * BR * ldb * 2) : 0u,
          0, 0);
  };

  wfloatx16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.f;
  struct Frags {
    wbf16x8_t a[2], b[2];
  };
  Frags f[2];
  auto read = [&](Frags& d, const char* a, const char* b, int k) {
#pragma unroll
    for (int i = 0; i < 2; ++i) d.a[i] = wfrag(a, wp * 64 + i * 32, k, lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) d.b[j] = wfrag(b, wq * 64 + j * 32, k, lane);
  };
  auto mfma = [&](const Frags& d) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d.a[i], d.b[j], acc[i][j], 0, 0, 0);
  };
  auto sched = [&]() {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Chunk c is in (a, b); chunk c+1's X is on its way to bn, its dZ in reg.
  auto chunk = [&](char* a, char* b, char* an, char* bn, int c) {
    read(f[1], a, b, 1);
    put(an, 0), put(an, 1), put(an, 2);
    mfma(f[0]);
    sched();
    read(f[0], a, b, 2);
    put(an, 3), put(an, 4), put(an, 5);
    mfma(f[1]);
    sched();
    read(f[1], a, b, 3);
    put(an, 6), put(an, 7);
    load(c + 2);
    mfma(f[0]);
    sched();
    // every load but the 8 just issued (X of chunk c+1 among them) and all LDS accesses done
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    request(b, c + 2);
    read(f[0], an, bn, 0);
    mfma(f[1]);
    __builtin_amdgcn_sched_barrier(0);
  };

  load(0);
  request(sb0, 0);
#pragma unroll
  for (int i = 0; i < 8; ++i) put(sa0, i);
  request(sb1, 1);
  load(1);
  if (BF) opt_prepare(ea.opt);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  read(f[0], sa0, sb0, 0);
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < nch; c += 2) {   // (a chunk past the end is zeros)
    chunk(sa0, sb0, sa1, sb1, c);
    chunk(sa1, sb1, sa0, sb0, c + 1);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  if (ea.with_db && ty == 0) {
    // bias gradient: the threads' column sums, added in thread order
    float* red = reinterpret_cast<float*>(sa0);   // [8][128]
#pragma unroll
    for (int k = 0; k < 4; ++k) red[ar * WT + ax + k] = dbs[k];
    __syncthreads();
    if (tid < WT && tid < np) {
      float s = red[tid];
#pragma unroll
      for (int g = 1; g < 8; ++g) s = __fadd_rn(s, red[g * WT + tid]);
      bias_epilogue<EPI>(ea, p0 + tid, s);
    }
  }

  // Epilogue from the accumulators, as above.
  const int c32 = lane & 31, r4 = (lane >> 5) * 4;
  const int prow = p0 + wp * 64, qcol = q0 + wq * 64;
  const int nrow = min(64, pr.P - prow), ncol = min(64, pr.Q - qcol);
  if (nrow <= 0 || ncol <= 0) return;
  const int64_t ld = ea.ldo;
  const int64_t org = (int64_t)prow * ld + qcol;
  const int64_t end = (int64_t)(nrow - 1) * ld + ncol;
  auto desc = [&](const float* t) { return make_rsrc(t ? t + org : nullptr, t ? (int)(end * 4) : 0); };
  const bool two = ea.opt.kind != OF_OPT_SGD;
  const rsrc_t ro = desc(BF ? ea.W.w : ea.out);
  const rsrc_t rm = BF ? desc(ea.W.m) : ro, rv = BF ? desc(two ? ea.W.v : nullptr) : ro;
  const rsrc_t rg = BF ? desc(ea.gW) : ro;
  const rsrc_t rs = BF && ea.W.w_bf16 ? make_rsrc(ea.W.w_bf16 + org, (int)(end * 2)) : ro;
  auto at = [&](int t, int k) -> uint32_t {   // element of register k of block t = 2 i + j
    const int col = (t & 1) * 32 + c32;
    return col < ncol ? (uint32_t)(((t >> 1) * 32 + (k >> 2) * 8 + r4 + (k & 3)) * ld + col) : kOOB / 4;
  };
  float w[2][16], m[2][16], v[2][16];
  auto fetch = [&](int t) {
    if constexpr (BF) {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        w[t & 1][k] = bload1(ro, at(t, k) * 4);
        m[t & 1][k] = bload1(rm, at(t, k) * 4);   // no m: 0
        v[t & 1][k] = bload1(rv, at(t, k) * 4);
      }
    }
  };
  const bool pair = BF && ea.W.w_bf16 && ld % 2 == 0 && ((uintptr_t)ea.W.w_bf16 & 3u) == 0 &&
                    (ncol & 1) == 0;
  auto st = [&](const rsrc_t& r, uint32_t off, float x) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, off, 0, 0);
  };
  fetch(0);
  auto block = [&](auto T_) {
    constexpr int t = decltype(T_)::value;
    if constexpr (t + 1 < 4) fetch(t + 1);
    float g[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) g[k] = acc[t >> 1][t & 1][k];
    if (BF ? ea.gW != nullptr : ea.accumulate != 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) g[k] = __fadd_rn(bload1(rg, at(t, k) * 4), g[k]);
    }
    if constexpr (!BF) {
#pragma unroll
      for (int k = 0; k < 16; ++k) st(ro, at(t, k) * 4, g[k]);
    } else {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        opt_update(ea.opt, w[t & 1][k], g[k], m[t & 1][k], v[t & 1][k]);
        st(ro, at(t, k) * 4, w[t & 1][k]);
        st(rm, at(t, k) * 4, m[t & 1][k]);   // no m: dropped
        if (two) st(rv, at(t, k) * 4, v[t & 1][k]);
      }
      if (pair) {   // lanes 2l and 2l+1 trade a value: two columns of a row each
        const bool odd = lane & 1;
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          const float mine = odd ? w[t & 1][k + 1] : w[t & 1][k], give = odd ? w[t & 1][k] : w[t & 1][k + 1];
          const float got = __int_as_float(
              __builtin_amdgcn_mov_dpp(__float_as_int(give), 0xb1, 0xf, 0xf, true));
          const uint32_t e = at(t, k);
          __builtin_amdgcn_raw_buffer_store_b32(odd ? cvt2(got, mine) : cvt2(mine, got), rs,
                                                e == kOOB / 4 ? kOOB : (e + (odd ? (uint32_t)ld - 1u : 0u)) * 2u,
                                                0, 0);
        }
      } else if (ea.W.w_bf16) {
#pragma unroll
        for (int k = 0; k < 16; ++k)
          __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(w[t & 1][k]), rs,
                                                at(t, k) == kOOB / 4 ? kOOB : at(t, k) * 2u, 0, 0);
      }
    }
  };
  each(std::make_integer_sequence<int, 4>{}, block);
}

hipError_t wgrad_bf16_launch(int kind, const GemmProblem& pr, const EpiArgs& ea, hipStream_t s) {
  const dim3 g((pr.P + WT - 1) / WT, (pr.Q + WT - 1) / WT);
  if (kind == EPI_WGRAD) hipLaunchKernelGGL((wgrad_bf16_kernel<EPI_WGRAD>), g, dim3(256), 0, s, pr, ea);
  else if (kind == EPI_WGRAD_BF) hipLaunchKernelGGL((wgrad_bf16_kernel<EPI_WGRAD_BF>), g, dim3(256), 0, s, pr, ea);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int EPI, bool A32, int ACT>
static hipError_t launch(const GemmProblem& pr, const EpiArgs& ea, int S, int r_split, int cz,
                         hipStream_t s) {
  const dim3 g((pr.P + BT - 1) / BT, (pr.Q + BT - 1) / BT, S + cz);
  if (ea.res)
    hipLaunchKernelGGL((gemm_bf16_wide_kernel<EPI, A32, ACT, true>), g, dim3(256), 0, s, pr, ea, r_split);
  else
    hipLaunchKernelGGL((gemm_bf16_wide_kernel<EPI, A32, ACT, false>), g, dim3(256), 0, s, pr, ea, r_split);
  return hipGetLastError();
}

// S > 1 (a forward only): the sums of each split to ws, [S][P][Q]; the caller adds them.
hipError_t gemm_bf16_wide_launch(int kind, const GemmProblem& pr, const EpiArgs& ea_in, int S,
                                 int r_split, int cz, void* ws, hipStream_t s) {
  EpiArgs ea = ea_in;
  if (S > 1) {
    if (kind != EPI_FWD || ws == nullptr) return hipErrorInvalidValue;
    ea.out = (float*)ws;
    ea.ldo = pr.Q;
    ea.yb = nullptr;
    ea.z = nullptr;
    ea.bias = nullptr;
    ea.res = nullptr;
    ea.act = OF_ACT_NONE;
  }
  if (kind == EPI_FWD)   // (the forward's activation needs no loads: chosen in the kernel)
    return pr.a_bf16 ? launch<EPI_FWD, false, OF_ACT_NONE>(pr, ea, S, r_split, cz, s)
                     : launch<EPI_FWD, true, OF_ACT_NONE>(pr, ea, S, r_split, cz, s);
  if (kind != EPI_DGRAD) return hipErrorInvalidValue;
  switch (ea.act) {
    case OF_ACT_RELU: return launch<EPI_DGRAD, true, OF_ACT_RELU>(pr, ea, S, r_split, cz, s);
    case OF_ACT_GELU: return launch<EPI_DGRAD, true, OF_ACT_GELU>(pr, ea, S, r_split, cz, s);
    default: return launch<EPI_DGRAD, true, OF_ACT_NONE>(pr, ea, S, r_split, cz, s);
  }
}

}  // namespace opfuse

// Forward and data gradient of tall products with a short reduction (a 1x1
// convolution as a linear layer over 16k to 400k pixel rows, at most 64
// reduction elements onto at most 256 channels).
//
// Memory bounds them: reading X (or dZ) and writing the output is all there is.
// The tiled kernel fetches a row panel once per column tile and spends a
// workgroup's life on one or two chunks, a barrier and an LDS round trip; here W
// stays in LDS, a wavefront walks panels of 32 rows, holds a panel's operands in
// registers (the next panel's are in flight), and stores every 32x32 block straight
// from the accumulators: no barrier after the start.  The stores bypass the
// caches (tens of megabytes that nothing reads soon); with ordinary ones this was no
// faster than the tiles (42 against 40 us for 100352 x 24 -> 144), with them that
// layer's forward, backward and update went from 98 to 88 us.
//
// v_mfma_f32_32x32x2_f32 takes the reduction in the tiled kernel's order, two
// elements a step from 0, so results are the same bit for bit (the fused and the
// plain forward may run on different kernels).

#include <algorithm>

#include "gemm_common.h"

namespace opfuse {

typedef float rfloatx16_t __attribute__((ext_vector_type(16)));

// RS: MFMA steps (2 RS >= R; what is past R multiplies zeros).
template <int EPI, int RS>
__global__ __launch_bounds__(256) void gemm_rows_kernel(GemmProblem pr, EpiArgs ea) {
  static_assert(EPI == EPI_FWD || EPI == EPI_DGRAD, "forward and data gradient only");
  constexpr int LDW = 2 * RS + 1;
  extern __shared__ float ws[];   // W as [q][r], rows of LDW
  if constexpr (EPI == EPI_FWD) {
    if ((int)blockIdx.z < ea.carry.cz) {
      carry_update(ea.carry);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
  const int nb = (pr.Q + 31) / 32;
  for (int i = tid; i < nb * 32 * 2 * RS; i += 256) {
    // (along W's contiguous index)
    const int q = EPI == EPI_FWD ? i / (2 * RS) : i % (nb * 32);
    const int r = EPI == EPI_FWD ? i % (2 * RS) : i / (nb * 32);
    ws[q * LDW + r] = q < pr.Q && r < pr.R ? pr.B[q * pr.b_sq + r * pr.b_sr] : 0.f;
  }
  __syncthreads();

  const int np = (pr.P + 31) / 32, stride = gridDim.x * 4;
  auto load = [&](float (&a)[RS], int panel) {
    const bool ok = panel < np && panel * 32 + c < pr.P;
    const rsrc_t ra = make_rsrc(pr.A + (int64_t)(panel < np ? panel : 0) * 32 * pr.a_sp);
#pragma unroll
    for (int s = 0; s < RS; ++s)
      a[s] = bload1(ra, ok && 2 * s + h < pr.R ? (uint32_t)((c * pr.a_sp + 2 * s + h) * 4) : kOOB);
  };
  float a[RS], an[RS];
  int panel = blockIdx.x * 4 + (tid >> 6);
  load(a, panel);
  for (; panel < np; panel += stride) {
    load(an, panel + stride);
    const int p0 = panel * 32;
    auto at = [&](int64_t ld, int k, int j) -> uint32_t {   // register k of column block j
      const int p = (k >> 2) * 8 + h * 4 + (k & 3);
      return p0 + p < pr.P && j * 32 + c < pr.Q ? (uint32_t)((p * ld + j * 32 + c) * 4) : kOOB;
    };
    const rsrc_t ro = make_rsrc(ea.out + (int64_t)p0 * ea.ldo);
    const rsrc_t rz = EPI == EPI_FWD && ea.z ? make_rsrc(ea.z + (int64_t)p0 * ea.ldz) : ro;
    const bool dact = EPI == EPI_DGRAD && ea.act != OF_ACT_NONE;
    const rsrc_t rp = dact ? make_rsrc(ea.prev + (int64_t)p0 * ea.ldp) : ro;
    const rsrc_t rr = ea.res ? make_rsrc(ea.res + (int64_t)p0 * ea.ldr) : ro;
    for (int j = 0; j < nb; ++j) {
      float sv[16], rs[16];   // requested before the MFMAs, which hide them
      if (dact) {
#pragma unroll
        for (int k = 0; k < 16; ++k) sv[k] = bload1(rp, at(ea.ldp, k, j));
      }
      if (ea.res) {
#pragma unroll
        for (int k = 0; k < 16; ++k) rs[k] = bload1(rr, at(ea.ldr, k, j));
      }
      const float bias = EPI == EPI_FWD && ea.bias && j * 32 + c < pr.Q ? ea.bias[j * 32 + c] : 0.f;
      rfloatx16_t acc;
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[k] = 0.f;
#pragma unroll
      for (int s = 0; s < RS; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], ws[(j * 32 + c) * LDW + 2 * s + h], acc, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        float v = acc[k];
        if constexpr (EPI == EPI_FWD) {
          if (ea.bias) v = __fadd_rn(v, bias);
          if (ea.z) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rz, at(ea.ldz, k, j), 0, 2);
          v = act_fwd(ea.act, v);
        } else if (dact) {
          v = __fmul_rn(v, act_grad(ea.act, sv[k]));
        }
        if (ea.res) v = __fadd_rn(v, rs[k]);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ro, at(ea.ldo, k, j), 0, 2);
      }
    }
#pragma unroll
    for (int s = 0; s < RS; ++s) a[s] = an[s];
  }
}

template <int RS>
static hipError_t launch_rs(int kind, const GemmProblem& pr, const EpiArgs& ea, int cz, hipStream_t s) {
  const int wgs = (int)std::min<int64_t>(1024, ((int64_t)pr.P + 127) / 128);
  const dim3 grid(wgs, 1, 1 + cz);
  const size_t lds = (size_t)((pr.Q + 31) / 32) * 32 * (2 * RS + 1) * sizeof(float);
  if (kind == EPI_FWD)
    hipLaunchKernelGGL((gemm_rows_kernel<EPI_FWD, RS>), grid, dim3(256), lds, s, pr, ea);
  else
    hipLaunchKernelGGL((gemm_rows_kernel<EPI_DGRAD, RS>), grid, dim3(256), lds, s, pr, ea);
  return hipGetLastError();
}

static int steps_of(int R) { return R <= 16 ? 8 : R <= 24 ? 12 : R <= 32 ? 16 : 32; }

// At least 16384 rows onto 33 to 256 columns with at most 64 reduction elements,
// fp32 and strided: where the tiled kernels take whole reductions in the same
// order.  W takes at most 48 KB of LDS.
bool gemm_rows_ok(int kind, const GemmProblem& pr, const EpiArgs& ea) {
  if ((kind != EPI_FWD && kind != EPI_DGRAD) || pr.conv || ea.yb || pr.a_sr != 1) return false;
  for (int64_t ld : {pr.a_sp, ea.ldo, ea.ldz, ea.ldp, ea.ldr})
    if (ld > (1 << 22)) return false;   // 32-bit offsets within a panel
  return pr.P >= 16384 && pr.Q > 32 && pr.Q <= 256 && pr.R <= 64 &&
         (pr.Q + 31) / 32 * 32 * (2 * steps_of(pr.R) + 1) <= 12288;
}

hipError_t gemm_rows_launch(int kind, const GemmProblem& pr, const EpiArgs& ea_in, hipStream_t s) {
  EpiArgs ea = ea_in;
  const int64_t wgs = std::min<int64_t>(1024, ((int64_t)pr.P + 127) / 128);
  ea.carry.cz = ea.carry.t[0].p.w ? carry_slices(ea.carry, wgs) : 0;
  switch (steps_of(pr.R)) {
    case 8: return launch_rs<8>(kind, pr, ea, ea.carry.cz, s);
    case 12: return launch_rs<12>(kind, pr, ea, ea.carry.cz, s);
    case 16: return launch_rs<16>(kind, pr, ea, ea.carry.cz, s);
    default: return launch_rs<32>(kind, pr, ea, ea.carry.cz, s);
  }
}

}  // namespace opfuse

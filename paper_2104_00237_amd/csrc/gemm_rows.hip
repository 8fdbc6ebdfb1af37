// Forward of tall products with a short reduction onto more output than the caches
// hold (a 1x1 convolution as a linear layer over 400k pixel rows, at most 64 reduction
// elements onto at most 256 channels).
//
// Memory bounds them: reading X and writing the output is all there is.  The tiled
// kernel fetches a row panel once per column tile and spends a workgroup's life on
// one or two chunks, a barrier and an LDS round trip; here W stays in LDS, a wavefront
// walks panels of 32 rows, holds a panel's operands in registers (the next panel's
// are in flight), and stores every 32x32 block straight from the accumulators: no
// barrier after the start.
//
// The stores bypass the caches, and that is most of the gain (with ordinary ones
// 100352 x 24 -> 144 takes 42 us, 40 on the tiles).  The next layer reads the output at
// once, so it must be too large to wait in a cache: MobileNetV2's step at batch 32 takes
// 2.94 ms without this kernel, 2.91 with outputs of 128 MB and more on it (401408 x 16
// -> 96), 2.97 with only the smaller ones on it, although these layers alone are faster
// (100352 x 24 -> 144 with its backward and update 98 -> 88 us), and 2.99 with data
// gradients on it as well.
//
// v_mfma_f32_32x32x2_f32 takes the reduction in the tiled kernel's order, two
// elements a step from 0, so results are the same bit for bit (the fused and the
// plain forward run on different kernels).

#include <algorithm>

#include "gemm_common.h"

namespace opfuse {

typedef float rfloatx16_t __attribute__((ext_vector_type(16)));

// RS: MFMA steps (2 RS >= R; what is past R multiplies zeros).
template <int RS>
__global__ __launch_bounds__(256) void gemm_rows_kernel(GemmProblem pr, EpiArgs ea) {
  constexpr int LDW = 2 * RS + 1;
  extern __shared__ float ws[];   // W as [q][r], rows of LDW
  if ((int)blockIdx.z < ea.carry.cz) {
    carry_update(ea.carry);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
  const int nb = (pr.Q + 31) / 32;
  for (int i = tid; i < nb * 32 * 2 * RS; i += 256) {
    const int q = i / (2 * RS), r = i % (2 * RS);
    ws[q * LDW + r] = q < pr.Q && r < pr.R ? pr.B[q * pr.b_sq + r] : 0.f;
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
    const rsrc_t rz = ea.z ? make_rsrc(ea.z + (int64_t)p0 * ea.ldz) : ro;
    const rsrc_t rr = ea.res ? make_rsrc(ea.res + (int64_t)p0 * ea.ldr) : ro;
    for (int j = 0; j < nb; ++j) {
      float rs[16];   // requested before the MFMAs, which hide them
      if (ea.res) {
#pragma unroll
        for (int k = 0; k < 16; ++k) rs[k] = bload1(rr, at(ea.ldr, k, j));
      }
      const float bias = ea.bias && j * 32 + c < pr.Q ? ea.bias[j * 32 + c] : 0.f;
      rfloatx16_t acc;
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[k] = 0.f;
#pragma unroll
      for (int s = 0; s < RS; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], ws[(j * 32 + c) * LDW + 2 * s + h], acc, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        float v = acc[k];
        if (ea.bias) v = __fadd_rn(v, bias);
        if (ea.z) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rz, at(ea.ldz, k, j), 0, 2);
        v = act_fwd(ea.act, v);
        if (ea.res) v = __fadd_rn(v, rs[k]);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ro, at(ea.ldo, k, j), 0, 2);
      }
    }
#pragma unroll
    for (int s = 0; s < RS; ++s) a[s] = an[s];
  }
}

template <int RS>
static hipError_t launch_rs(const GemmProblem& pr, const EpiArgs& ea, int cz, hipStream_t s) {
  const int wgs = (int)std::min<int64_t>(1024, ((int64_t)pr.P + 127) / 128);
  const dim3 grid(wgs, 1, 1 + cz);
  const size_t lds = (size_t)((pr.Q + 31) / 32) * 32 * (2 * RS + 1) * sizeof(float);
  hipLaunchKernelGGL((gemm_rows_kernel<RS>), grid, dim3(256), lds, s, pr, ea);
  return hipGetLastError();
}

static int steps_of(int R) { return R <= 16 ? 8 : R <= 24 ? 12 : R <= 32 ? 16 : 32; }

// At least 128 MB of output in 33 to 256 columns (so 131072 rows or more) with at most
// 64 reduction elements, fp32 and strided: where the tiled kernels take whole
// reductions in the same order.  W takes at most 48 KB of LDS.
bool gemm_rows_ok(int kind, const GemmProblem& pr, const EpiArgs& ea) {
  if (kind != EPI_FWD || pr.conv || ea.yb || pr.a_sr != 1 || pr.b_sr != 1) return false;
  for (int64_t ld : {pr.a_sp, ea.ldo, ea.ldz, ea.ldr})
    if (ld > (1 << 22)) return false;   // 32-bit offsets within a panel
  return (int64_t)pr.P * pr.Q >= (1 << 25) && pr.Q > 32 && pr.Q <= 256 && pr.R <= 64 &&
         (pr.Q + 31) / 32 * 32 * (2 * steps_of(pr.R) + 1) <= 12288;
}

hipError_t gemm_rows_launch(const GemmProblem& pr, const EpiArgs& ea_in, hipStream_t s) {
  EpiArgs ea = ea_in;
  const int64_t wgs = std::min<int64_t>(1024, ((int64_t)pr.P + 127) / 128);
  ea.carry.cz = ea.carry.t[0].p.w ? carry_slices(ea.carry, wgs) : 0;
  switch (steps_of(pr.R)) {
    case 8: return launch_rs<8>(pr, ea, ea.carry.cz, s);
    case 12: return launch_rs<12>(pr, ea, ea.carry.cz, s);
    case 16: return launch_rs<16>(pr, ea, ea.carry.cz, s);
    default: return launch_rs<32>(pr, ea, ea.carry.cz, s);
  }
}

}  // namespace opfuse

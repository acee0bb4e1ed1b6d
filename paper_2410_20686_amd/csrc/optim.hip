// Training step around the rasterizer: the L1 image loss with its gradient, and one Adam update
// of the Gaussian parameters kept before their activations (the 3DGS recipe the paper trains
// with, per its implementation details: scale = exp(raw), opacity = sigmoid(raw), quaternions
// normalised inside the rasterizer).  Both are streaming passes bound by HBM bandwidth.
#include <mutex>

#include "common.h"

namespace odgs {

// Scratch of odgs_l1_loss_noalloc: the per-block partial sums of l1_kernel, kept in a file-scope
// device array so that entry point allocates nothing.  Every GPU the library runs on holds its own
// copy at its own address until the process ends.  In host code `scratch` names a host-side
// stand-in, not device memory: kernels get the address hipGetSymbolAddress returns for the current
// device (l1_scratch_ptr), never the array's name.
constexpr int kL1ScratchBlocks = 65536;  // 512 KiB of doubles
static __device__ __align__(256) double scratch[kL1ScratchBlocks];

namespace {

constexpr int kL1Threads = 256;
constexpr int kL1Ipt = 16;
constexpr int kL1Block = kL1Threads * kL1Ipt;

// dL/drgb = sign(rgb - target) / count (sign(0) = 0) and per-block sums of |rgb - target| in
// double (summed in a fixed order by the final kernel, so the loss is reproducible).
__global__ __launch_bounds__(kL1Threads) void l1_kernel(const float* __restrict__ rgb, const float* __restrict__ tgt,
                                                       int64_t count, float inv_count, float* __restrict__ dL,
                                                       double* __restrict__ partial) {
  __shared__ double wsum[kL1Threads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kL1Block;
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < kL1Ipt; ++r) {
    const int64_t i = base + r * kL1Threads + threadIdx.x;  // coalesced
    if (i < count) {
      const float d = rgb[i] - tgt[i];
      dL[i] = d > 0.0f ? inv_count : (d < 0.0f ? -inv_count : 0.0f);
      s += (double)fabsf(d);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kL1Threads / kWave; ++w) t += wsum[w];
    partial[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(256) void l1_final_kernel(const double* __restrict__ partial, int nblocks,
                                                       double inv_count, float* __restrict__ loss) {
  __shared__ double wsum[4];
  double s = 0.0;
#pragma unroll 8
  for (int b = threadIdx.x; b < nblocks; b += 256) s += partial[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) loss[0] = (float)(((wsum[0] + wsum[1]) + (wsum[2] + wsum[3])) * inv_count);
}

enum Act { kIdentity = 0, kExp = 1, kSigmoid = 2 };

struct AdamArgs {
  float beta1, beta2, eps;
};

// One parameter array: lr[g0] for elements below `split`, lr[g1] above it (the SH DC planes vs the rest).
struct AdamArray {
  float *raw, *act;
  const float* grad;
  float *m, *v;
  int64_t count, split;
  int32_t g0, g1, kind;
  uint32_t block0;  // first block of the array's elements
};
constexpr int kAdamArrays = 5;
constexpr int kAdamThreads = 256;
constexpr int kAdamBlock = 4 * kAdamThreads;  // elements
struct AdamTable {
  AdamArray a[kAdamArrays];
};

// The rates divided by the first bias correction, and the root of the second.
struct AdamRates {
  float r0, r1, root2;
};

template <int ACT>
__device__ inline void adam_element(float& raw, float& act, float grad, float& m, float& v, float rate, float root2,
                                    const AdamArgs& a) {
  float g = grad;
  if (ACT == kExp) g *= act;
  if (ACT == kSigmoid) g *= act * (1.0f - act);
  const float mm = a.beta1 * m + (1.0f - a.beta1) * g;
  const float vv = a.beta2 * v + (1.0f - a.beta2) * (g * g);
  const float p = raw - rate * mm / (sqrtf(vv) / root2 + a.eps);
  m = mm;
  v = vv;
  raw = p;
  act = ACT == kExp ? expf(p) : (ACT == kSigmoid ? 1.0f / (1.0f + expf(-p)) : p);
}

// Four elements of an array: neighbours from i on with VEC, else i and every kAdamThreads-th after it.
template <int ACT, bool VEC>
__device__ inline void adam_block(const AdamArray& q, int64_t i, const AdamRates& rates, const AdamArgs& a) {
  if (VEC && i + 4 <= q.count) {
    float4 raw = *reinterpret_cast<const float4*>(q.raw + i), m = *reinterpret_cast<const float4*>(q.m + i);
    float4 v = *reinterpret_cast<const float4*>(q.v + i), act = make_float4(0, 0, 0, 0);
    const float4 g = *reinterpret_cast<const float4*>(q.grad + i);
    if (ACT != kIdentity) act = *reinterpret_cast<const float4*>(q.act + i);
    adam_element<ACT>(raw.x, act.x, g.x, m.x, v.x, i < q.split ? rates.r0 : rates.r1, rates.root2, a);
    adam_element<ACT>(raw.y, act.y, g.y, m.y, v.y, i + 1 < q.split ? rates.r0 : rates.r1, rates.root2, a);
    adam_element<ACT>(raw.z, act.z, g.z, m.z, v.z, i + 2 < q.split ? rates.r0 : rates.r1, rates.root2, a);
    adam_element<ACT>(raw.w, act.w, g.w, m.w, v.w, i + 3 < q.split ? rates.r0 : rates.r1, rates.root2, a);
    *reinterpret_cast<float4*>(q.raw + i) = raw;
    *reinterpret_cast<float4*>(q.m + i) = m;
    *reinterpret_cast<float4*>(q.v + i) = v;
    *reinterpret_cast<float4*>(q.act + i) = act;
    return;
  }
  for (int e = 0; e < 4 && i < q.count; ++e, i += VEC ? 1 : kAdamThreads) {
    float raw = q.raw[i], act = ACT != kIdentity ? q.act[i] : 0.0f, m = q.m[i], v = q.v[i];
    adam_element<ACT>(raw, act, q.grad[i], m, v, i < q.split ? rates.r0 : rates.r1, rates.root2, a);
    q.raw[i] = raw;
    q.m[i] = m;
    q.v[i] = v;
    q.act[i] = act;
  }
}

// One Adam update per element (Kingma & Ba, with PyTorch's placement of eps): the gradient with
// respect to the activated value is chained through the activation (using the activated value
// the step's forward pass read), the moments updated, the raw parameter moved, and the activated
// value rewritten for the next forward pass.  The step count is read on the device.
//
// Bound by HBM: 32 bytes per element.  One launch over the five arrays; one thread per block raises the
// betas to the step's power, and a thread takes four elements, in words of 16 bytes with VEC (arrays so
// aligned): 72 us for 14.75M elements (250k Gaussians at SH degree 3), 130 us in five launches of one element
// per thread, each raising the betas for itself.  (One element per thread in one launch would also pass the
// 2^32 threads of a launch from 73M Gaussians on, which five launches took.)
template <bool VEC>
__global__ __launch_bounds__(kAdamThreads) void adam_kernel(AdamTable table, const float* __restrict__ lr,
                                                            const int32_t* __restrict__ step, AdamArgs a) {
  __shared__ AdamRates rates;
  int k = 0;
#pragma unroll
  for (int j = 1; j < kAdamArrays; ++j) k = blockIdx.x >= table.a[j].block0 ? j : k;
  const AdamArray& q = table.a[k];
  if (threadIdx.x == 0) {
    const float t = (float)(step[0] + 1);
    const float bc1 = 1.0f - powf(a.beta1, t), bc2 = 1.0f - powf(a.beta2, t);
    rates = AdamRates{lr[q.g0] / bc1, lr[q.g1] / bc1, sqrtf(bc2)};
  }
  __syncthreads();
  const int64_t i = (int64_t)(blockIdx.x - q.block0) * kAdamBlock + threadIdx.x * (VEC ? 4 : 1);
  if (q.kind == kExp)
    adam_block<kExp, VEC>(q, i, rates, a);
  else if (q.kind == kSigmoid)
    adam_block<kSigmoid, VEC>(q, i, rates, a);
  else
    adam_block<kIdentity, VEC>(q, i, rates, a);
}

__global__ void step_increment_kernel(int32_t* __restrict__ step) {
  if (threadIdx.x == 0) step[0] = step[0] + 1;
}

inline int l1_blocks(int64_t count) { return (int)((count + kL1Block - 1) / kL1Block); }

// Device address of `scratch` on the current device, looked up once per device (with that device
// current) on its first use and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

hipError_t l1_scratch_ptr(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

int64_t l1_noalloc_max_count() { return (int64_t)kL1ScratchBlocks * kL1Block; }

size_t l1_workspace_bytes(int64_t count) {
  return (((size_t)l1_blocks(count) * sizeof(double) + 255) / 256) * 256 + 256;
}

hipError_t launch_l1(const float* rgb, const float* tgt, int64_t count, float* dL, float* loss, void* ws,
                     hipStream_t st) {
  const int nb = l1_blocks(count);
  double* partial = static_cast<double*>(ws);
  if (nb > 0)
    hipLaunchKernelGGL(l1_kernel, dim3(nb), dim3(kL1Threads), 0, st, rgb, tgt, count,
                       (float)(1.0 / (double)count), dL, partial);
  hipLaunchKernelGGL(l1_final_kernel, dim3(1), dim3(256), 0, st, partial, nb,
                     count > 0 ? 1.0 / (double)count : 0.0, loss);
  return hipGetLastError();
}

hipError_t launch_l1_noalloc(const float* rgb, const float* tgt, int64_t count, float* dL, float* loss,
                             hipStream_t st) {
  if (count > l1_noalloc_max_count()) return hipErrorInvalidValue;
  double* partial = nullptr;
  const hipError_t e = l1_scratch_ptr(&partial);
  if (e != hipSuccess) return e;
  // every block of l1_kernel writes its partial and l1_final_kernel reads exactly those, so the
  // array needs no clearing between calls
  return launch_l1(rgb, tgt, count, dL, loss, partial, st);
}

hipError_t launch_adam_step(int64_t n, int32_t sh_degree, const odgs_param_ptrs& raw, const odgs_param_ptrs& act,
                            const odgs_param_ptrs& grad, const odgs_param_ptrs& m, const odgs_param_ptrs& v,
                            const float* lr, int32_t* step, const odgs_adam_hyper& hp, hipStream_t st) {
  const AdamArgs a{hp.beta1, hp.beta2, hp.eps};
  const int64_t K = (int64_t)(sh_degree + 1) * (sh_degree + 1);
  auto array = [](float* r, float* ac, const float* g, float* mm, float* vv, int64_t count, int64_t split, int g0, int g1,
                  int kind) { return AdamArray{r, ac, g, mm, vv, count, split, g0, g1, kind, 0}; };
  AdamTable t{{array(raw.means, act.means, grad.means, m.means, v.means, 3 * n, 3 * n, 0, 0, kIdentity),
               array(raw.scales, act.scales, grad.scales, m.scales, v.scales, 3 * n, 3 * n, 1, 1, kExp),
               array(raw.quats, act.quats, grad.quats, m.quats, v.quats, 4 * n, 4 * n, 2, 2, kIdentity),
               array(raw.opacities, act.opacities, grad.opacities, m.opacities, v.opacities, n, n, 3, 3, kSigmoid),
               array(raw.sh, act.sh, grad.sh, m.sh, v.sh, 3 * K * n, 3 * n, 4, 5, kIdentity)}};
  uintptr_t low = 0;
  for (const AdamArray& q : t.a)
    low |= reinterpret_cast<uintptr_t>(q.raw) | reinterpret_cast<uintptr_t>(q.act) | reinterpret_cast<uintptr_t>(q.grad) |
           reinterpret_cast<uintptr_t>(q.m) | reinterpret_cast<uintptr_t>(q.v);
  const bool vec = (low & 15) == 0;
  int64_t blocks = 0;
  for (AdamArray& q : t.a) {
    q.block0 = (uint32_t)blocks;
    blocks += (q.count + kAdamBlock - 1) / kAdamBlock;
  }
  if (blocks > 0) {
    if (vec)
      hipLaunchKernelGGL(adam_kernel<true>, dim3((unsigned)blocks), dim3(kAdamThreads), 0, st, t, lr, step, a);
    else
      hipLaunchKernelGGL(adam_kernel<false>, dim3((unsigned)blocks), dim3(kAdamThreads), 0, st, t, lr, step, a);
  }
  hipLaunchKernelGGL(step_increment_kernel, dim3(1), dim3(64), 0, st, step);
  return hipGetLastError();
}

}  // namespace odgs

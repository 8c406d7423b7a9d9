// Attached passes (derivatives of the geometry): kernels and launchers.
#include <hip/hip_runtime.h>

#include "lt_path.h"

namespace lt {

#ifdef LT_COUNTERS
inline namespace counted {
#endif

#include "lt_attached.inc"

// The attached LRB-3 over a batch's instance table (see k_trace_batch).
template <int SC>
__global__ void __launch_bounds__(256, 2) k_lrb3_att_batch(const PassArgs* __restrict__ T, int n) {
  extern __shared__ int lds[];
  for (int i = 0; i < n; ++i) lrb3_att_run<false, SC>(table_ptr(T, i), lds);
}
// The two-kernel attached LRB-3 reading one table entry: batches run their
// large attached instances through this pair, as the single-instance call
// does (the hand-off buffer and pass 3's counters are in the entry; the
// arguments stay in the table, so a replayed graph reads each step's seeds).
template <int SC>
__global__ void __launch_bounds__(768, 3) k_lrb3_att_p2_entry(const PassArgs* __restrict__ T) {
  extern __shared__ int lds[];
  lrb3_att_p2_run<false, SC>(table_ptr(T, 0), lds);
}
template <int SC>
__global__ void __launch_bounds__(768, 3) k_lrb3_att_p3_entry(const PassArgs* __restrict__ T) {
  extern __shared__ int lds[];
  lrb3_att_p3_run<false, SC>(table_ptr(T, 0), lds);
}

__global__ void __launch_bounds__(256) k_frames(DevScene sc) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i <= sc.n_static) write_frame(sc, i);
}

#ifdef LT_COUNTERS
}  // namespace counted
#endif

// ---------------------------------------------------------------- launchers
hipError_t launch_frames(const DevScene& sc, hipStream_t s) {
  hipLaunchKernelGGL(k_frames, dim3(sc.n_static / 256 + 1), dim3(256), 0, s, sc);
  return hipGetLastError();
}
static size_t stack_bytes(const PassArgs& A, int block) { return (size_t)A.sc.stack_n * block * sizeof(int); }
static size_t hgrad_bytes(const PassArgs& A) {
  return A.hgrad_lds ? (size_t)A.sc.hf_G * A.sc.hf_G * sizeof(float) : 0;
}
static size_t agrad_bytes(const PassArgs& A) { return A.agrad_lds ? (size_t)A.n_texels * 3 * sizeof(float) : 0; }

hipError_t set_lds_limit_att(int bytes) {
  for (const void* f : {(const void*)k_lrb3_att<false, 1>, (const void*)k_lrb3_att<false, 3>, (const void*)k_lrb3_att<true, 1>,
                        (const void*)k_lrb3_att<true, 3>, (const void*)k_reslrb_att<false, 1>,
                        (const void*)k_reslrb_att<false, 3>, (const void*)k_reslrb_att<true, 1>,
                        (const void*)k_reslrb_att<true, 3>, (const void*)k_naive_att_bwd<false>,
                        (const void*)k_naive_att_bwd<true>, (const void*)k_lrb3_att_batch<1 | kScBatch>,
                        (const void*)k_lrb3_att_batch<1 | kScAny | kScBatch>, (const void*)k_lrb3_att_p2_entry<1>,
                        (const void*)k_lrb3_att_p2_entry<3>, (const void*)k_lrb3_att_p3_entry<1>,
                        (const void*)k_lrb3_att_p3_entry<3>, (const void*)k_lrb3_att_p2<false, 1>,
                        (const void*)k_lrb3_att_p2<false, 3>, (const void*)k_lrb3_att_p2<true, 1>,
                        (const void*)k_lrb3_att_p2<true, 3>, (const void*)k_lrb3_att_p3<false, 1>,
                        (const void*)k_lrb3_att_p3<false, 3>, (const void*)k_lrb3_att_p3<true, 1>,
                        (const void*)k_lrb3_att_p3<true, 3>}) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

const void* att_kernel(BwdKernel k) {
  switch (k) {
    case BwdKernel::naive_att: return (const void*)k_naive_att_bwd<false>;
    case BwdKernel::reslrb_att: return (const void*)k_reslrb_att<false, 1>;
    case BwdKernel::lrb3_att: return (const void*)k_lrb3_att<false, 1>;
    case BwdKernel::lrb3_att_cond: return (const void*)k_lrb3_att<true, 1>;
    case BwdKernel::lrb3_att_batch: return (const void*)k_lrb3_att_batch<1 | kScBatch>;
    case BwdKernel::lrb3_att_p2: return (const void*)k_lrb3_att_p2<false, 1>;
    case BwdKernel::lrb3_att_p3: return (const void*)k_lrb3_att_p3<false, 1>;
    case BwdKernel::lrb3_att_p3_cond: return (const void*)k_lrb3_att_p3<true, 1>;
    case BwdKernel::lrb3_att_p3_entry: return (const void*)k_lrb3_att_p3_entry<1>;
    default: return nullptr;
  }
}

#ifdef LT_COUNTERS
hipError_t add_counters_att(uint64_t* out, bool reset) {
  uint64_t v[16];
  hipError_t e = hipMemcpyFromSymbol(v, HIP_SYMBOL(lt_counters), sizeof(v), 0, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return e;
  for (int i = 0; i < 16; ++i) out[i] += v[i];
  if (!reset) return e;
  uint64_t z[16] = {0};
  return hipMemcpyToSymbol(HIP_SYMBOL(lt_counters), z, sizeof(z), 0, hipMemcpyHostToDevice);
}
#endif

hipError_t launch_lrb3_att(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL((A.cond ? k_lrb3_att<true, sc> : k_lrb3_att<false, sc>), dim3(grid), dim3(block), stack_bytes(A, block) + hgrad_bytes(A) + agrad_bytes(A), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_trace_att(const PassArgs& A, bool tape, bool resv, int grid, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    const size_t sh = stack_bytes(A, 256);
    if (tape && resv)
      hipLaunchKernelGGL((A.cond ? k_trace_att<true, true, true, sc> : k_trace_att<true, true, false, sc>), dim3(grid),
                         dim3(256), sh, s, A);
    else if (tape)
      hipLaunchKernelGGL((A.cond ? k_trace_att<true, false, true, sc> : k_trace_att<true, false, false, sc>), dim3(grid),
                         dim3(256), sh, s, A);
    else
      hipLaunchKernelGGL((A.cond ? k_trace_att<false, true, true, sc> : k_trace_att<false, true, false, sc>), dim3(grid),
                         dim3(256), sh, s, A);
  });
  return hipGetLastError();
}
hipError_t launch_naive_att_bwd(const PassArgs& A, int grid, hipStream_t s) {
  hipLaunchKernelGGL(A.cond ? k_naive_att_bwd<true> : k_naive_att_bwd<false>, dim3(grid), dim3(256), hgrad_bytes(A) + agrad_bytes(A), s, A);
  return hipGetLastError();
}
hipError_t launch_reslrb_att(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL((A.cond ? k_reslrb_att<true, sc> : k_reslrb_att<false, sc>), dim3(grid), dim3(block), stack_bytes(A, block) + hgrad_bytes(A) + agrad_bytes(A), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_lrb3_att_p2(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL((A.cond ? k_lrb3_att_p2<true, sc> : k_lrb3_att_p2<false, sc>), dim3(grid), dim3(block), stack_bytes(A, block), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_lrb3_att_p3(const PassArgs& A, int grid, int block, hipStream_t s) {
  by_scene_hf(scene_kind(A.sc), [&](auto sc) {
    hipLaunchKernelGGL((A.cond ? k_lrb3_att_p3<true, sc> : k_lrb3_att_p3<false, sc>), dim3(grid), dim3(block), stack_bytes(A, block) + hgrad_bytes(A) + agrad_bytes(A), s, A);
  });
  return hipGetLastError();
}
hipError_t launch_lrb3_att_batch(const PassArgs* table, int n, int kind, int stack_n, size_t grad_lds, int grid,
                                 hipStream_t s) {
  hipLaunchKernelGGL((kind & kScTree) ? k_lrb3_att_batch<1 | kScAny | kScBatch> : k_lrb3_att_batch<1 | kScBatch>, dim3(grid), dim3(256),
                     (size_t)stack_n * 256 * sizeof(int) + grad_lds, s, table, n);
  return hipGetLastError();
}
hipError_t launch_lrb3_att_split_entry(const PassArgs* entry, int kind, int stack_n, size_t grad_lds, int grid2, int grid3,
                                      int block3, hipStream_t s) {
  const size_t st2 = (size_t)stack_n * 256 * sizeof(int), st3 = (size_t)stack_n * block3 * sizeof(int);
  hipError_t e = hipSuccess;
  by_scene_hf(kind, [&](auto sc) {
    hipLaunchKernelGGL(k_lrb3_att_p2_entry<sc>, dim3(grid2), dim3(256), st2, s, entry);
    e = hipGetLastError();
    if (e != hipSuccess) return;
    hipLaunchKernelGGL(k_lrb3_att_p3_entry<sc>, dim3(grid3), dim3(block3), st3 + grad_lds, s, entry);
    e = hipGetLastError();
  });
  return e;
}

}  // namespace lt

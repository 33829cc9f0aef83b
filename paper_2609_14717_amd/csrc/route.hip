// Route: split each verified window by its accepted prefix (Eq. 1;
// Algorithm 1 "Given" and steps 5-6; greedy verification, Section 2
// "Preliminaries").
#include "co_route.h"

namespace co {

namespace {

constexpr int kRouteThreads = 1024;   // largest workgroup of a wide window

// One wavefront per sequence: drafted windows.
__global__ __launch_bounds__(64) void route_kernel(RouteArgs a) {
  route_sequence(a, blockIdx.x, threadIdx.x);
}

// One workgroup per sequence: windows of more than 64 rows (prompts, recorded
// responses), whose rows a single wavefront would take 64 at a time, each a
// dependent page-table read: the training forward (8 x 4096 rows, then 2048
// blocks) 226 -> 215 us, a 2048-row prompt 373 -> 370 us.
__global__ __launch_bounds__(kRouteThreads) void route_wide_kernel(RouteArgs a) {
  __shared__ int first[kRouteThreads / 64];
  const int s = blockIdx.x, t = threadIdx.x, nt = blockDim.x;
  const int B = a.B, p0 = a.ctx_len[s];   // read by every thread before the barriers below
  int m = B;
  if (!(a.flags & CO_ROUTE_ACCEPT_ALL)) {
    const bool bits = a.flags & CO_ROUTE_ACCEPT_BITS;
    const int32_t* dr = a.draft + static_cast<int64_t>(s) * B;
    const int32_t* tg = bits ? nullptr : a.target + static_cast<int64_t>(s) * B;
    for (int j = t; j < B; j += nt)
      if (bits ? dr[j] == 0 : dr[j] != tg[j]) {
        m = j;   // this thread's first
        break;
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o));
    if ((t & 63) == 0) first[t >> 6] = m;
    __syncthreads();
    for (int v = 0; v < (nt >> 6); ++v) m = min(m, first[v]);
  }
  int err = route_length_error(a, p0);   // uniform over the workgroup
  const bool look = err == 0 && !(a.flags & CO_ROUTE_CARRY_ONLY);
  if (__syncthreads_or(look && route_bad_page(a, s, p0, m, t, nt))) err = CO_ERR_PAGE_RANGE;
  route_write(a, s, p0, m, err, t, nt);
}

}  // namespace

hipError_t launch_route(const RouteArgs& a, hipStream_t stream) {
  if (a.S == 0) return hipSuccess;
  if (a.B <= 64) {
    hipLaunchKernelGGL(route_kernel, dim3(a.S), dim3(64), 0, stream, a);
  } else {
    const int threads = a.B >= kRouteThreads ? kRouteThreads : (a.B + 63) / 64 * 64;
    hipLaunchKernelGGL(route_wide_kernel, dim3(a.S), dim3(threads), 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace co

// Stochastic verification (T = 1): the acceptance decision and the correction
// or bonus draw of the standard speculative-sampling rule that Appendix A
// ("Why verification remains valid") relies on.  A proposal x ~ q at window
// position j is accepted with probability min(1, p_j(x) / q_j(x)); the first
// rejection at position m emits a token drawn from the normalised residual
// max(0, p_m - q_m); B acceptances emit a bonus drawn from p_B.
//
// Random draws arrive as 32-bit words, so the decisions are integer-exact:
//   * accept iff u * q(x) < p(x), u = (word >> 8) * 2^-24; the 24-bit by
//     24-bit product is exact in fp64, so this is the exact comparison;
//   * the draw uses fixed-point weights w(y) = floor(2^32 * d(y)) of the fp64
//     differences d(y) = p(y) - q(y) where positive (p(y) for a bonus, and for
//     a correction whose weights are all zero): y is the smallest token whose
//     running integer sum exceeds floor(word * W / 2^32), W the total weight.
//
// One workgroup of 1 to 16 wavefronts per sequence, by their number and the row's
// length (no scratch memory reaches this call, so a row's total is not summed
// across workgroups).  The first wavefront takes the acceptance decisions with one
// ballot per 64 positions.  Then the row of p (and q) is read once: every wavefront
// sums the weights of its own contiguous part, and only the part that holds the
// draw is read again for the running sums.  The row is bound by what one CU can
// keep in flight, so a lane has four 16-byte loads of each array outstanding (128
// KiB per workgroup of sixteen).  Integer sums: any order gives the same result.
// 32 sequences of 128000 tokens: 421 us with one load in flight per thread, 256
// threads and two passes, 20 us now.
#include "co_kernels.h"

namespace co {

namespace {

constexpr int kVerifyStep = 256;   // tokens of one wavefront load (four per lane)
constexpr int kVerifyDepth = 4;    // such loads in flight per array
constexpr int kFindPer = 8;        // tokens per thread and step of the draw's search

// Rows start at any multiple of four bytes (vocabularies need not be multiples
// of four, the arrays need not be 16-byte aligned); 16-byte global loads take
// such addresses.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint64_t weight_of(double d) {
  return d > 0.0 ? static_cast<uint64_t>(d * 4294967296.0) : 0ull;
}

__device__ __forceinline__ double difference(float p, float q) {
  return static_cast<double>(p) - static_cast<double>(q);
}

// The four weights of a load, w[k] of token k.  Below 1 (every probability but
// a certainty) floor(2^32 d) fits 32 bits: one conversion instead of the
// several of the 64-bit one.
__device__ __forceinline__ void weights4(f32x4u p, f32x4u q, uint64_t (&w)[4]) {
  double d[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) d[k] = difference(p[k], q[k]);
  if (__any(d[0] >= 1.0 || d[1] >= 1.0 || d[2] >= 1.0 || d[3] >= 1.0)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = weight_of(d[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = d[k] > 0.0 ? static_cast<uint32_t>(d[k] * 4294967296.0) : 0u;
  }
}

// Tokens y .. y + 3 of a row, zeros from `end` on.
__device__ __forceinline__ f32x4u load4(const float* r, int64_t y, int64_t end) {
  if (y + 4 <= end) return *reinterpret_cast<const f32x4u*>(r + y);
  f32x4u v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (y + k < end) v[k] = r[y + k];
  return v;
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int off) {
  const uint32_t lo = __shfl_up(static_cast<uint32_t>(v), off);
  const uint32_t hi = __shfl_up(static_cast<uint32_t>(v >> 32), off);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor(static_cast<uint32_t>(v), m);
  const uint32_t hi = __shfl_xor(static_cast<uint32_t>(v >> 32), m);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Tokens per wavefront: whole loads, so that only the row's end is ragged.
template <int NW>
__device__ __forceinline__ int wave_tokens(int V) {
  const int64_t unit = static_cast<int64_t>(NW) * kVerifyStep;
  return static_cast<int>((V + unit - 1) / unit) * kVerifyStep;
}

// Sum of the weights of this wavefront's part of the row, into red[wave].
template <bool HAS_Q>
__device__ void part_total(const float* p, const float* q, int V, int R, uint64_t* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lo = static_cast<int>(min(static_cast<int64_t>(V), static_cast<int64_t>(wave) * R));
  const int hi = static_cast<int>(min(static_cast<int64_t>(V), static_cast<int64_t>(lo) + R));
  const f32x4u zero = {0.f, 0.f, 0.f, 0.f};
  uint64_t s = 0;
  int n = (hi - lo) / kVerifyStep;   // whole loads
  const float* pp = p + lo + 4 * lane;
  const float* qp = HAS_Q ? q + lo + 4 * lane : nullptr;
  f32x4u pv[kVerifyDepth], qv[kVerifyDepth];
  for (; n >= kVerifyDepth; n -= kVerifyDepth) {
#pragma unroll
    for (int u = 0; u < kVerifyDepth; ++u) {
      pv[u] = *reinterpret_cast<const f32x4u*>(pp + u * kVerifyStep);
      qv[u] = HAS_Q ? *reinterpret_cast<const f32x4u*>(qp + u * kVerifyStep) : zero;
    }
#pragma unroll
    for (int u = 0; u < kVerifyDepth; ++u) {
      uint64_t w[4];
      weights4(pv[u], qv[u], w);
      s += (w[0] + w[1]) + (w[2] + w[3]);
    }
    pp += kVerifyDepth * kVerifyStep;
    if (HAS_Q) qp += kVerifyDepth * kVerifyStep;
  }
  for (int64_t y = pp - p; y - 4 * lane < hi; y += kVerifyStep) {
    uint64_t w[4];
    weights4(load4(p, y, hi), HAS_Q ? load4(q, y, hi) : zero, w);
    s += (w[0] + w[1]) + (w[2] + w[3]);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += shfl_xor_u64(s, m);
  if (lane == 0) red[wave] = s;
}

template <int NW>
__device__ uint64_t row_total(const float* p, const float* q, int V, int R, uint64_t* red) {
  __syncthreads();   // red[] may still be read from a previous use
  if (q) part_total<true>(p, q, V, R, red);
  else part_total<false>(p, q, V, R, red);
  __syncthreads();
  uint64_t W = 0;
#pragma unroll
  for (int v = 0; v < NW; ++v) W += red[v];
  return W;
}

// Smallest y with w(0) + ... + w(y) > t (t < the row's total weight), from the
// part totals in red[]: the part that holds it, then running sums over that part.
template <int NW>
__device__ int row_find(const float* p, const float* q, int V, int R, uint64_t t, uint64_t* red,
                        int* found) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t base = 0;
  int part = 0;
  while (part < NW - 1 && base + red[part] <= t) base += red[part++];
  const int64_t lo = static_cast<int64_t>(part) * R;
  const int64_t hi = min(static_cast<int64_t>(V), lo + R);
  if (tid == 0) *found = -1;
  const f32x4u zero = {0.f, 0.f, 0.f, 0.f};
  for (int64_t c0 = lo; c0 < hi; c0 += kFindPer * 64 * NW) {
    const int64_t y0 = c0 + kFindPer * tid;
    uint64_t w[kFindPer / 4][4], own = 0;
#pragma unroll
    for (int j = 0; j < kFindPer / 4; ++j) {
      const bool in = y0 + 4 * j < hi;
      const int64_t y = in ? y0 + 4 * j : 0, end = in ? hi : 0;
      weights4(load4(p, y, end), q ? load4(q, y, end) : zero, w[j]);
      own += (w[j][0] + w[j][1]) + (w[j][2] + w[j][3]);
    }
    uint64_t inc = own;   // inclusive scan within the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t o = shfl_up_u64(inc, off);
      if (lane >= off) inc += o;
    }
    __syncthreads();   // red[] and *found of the step before are read
    if (lane == 63) red[wave] = inc;
    __syncthreads();
    uint64_t before = base, total = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      if (v < wave) before += red[v];
      total += red[v];
    }
    before += inc - own;   // exclusive prefix of this thread's first token
    if (before <= t && t < before + own) {
      uint64_t c = before;
#pragma unroll
      for (int k = 0; k < kFindPer; ++k) {
        c += w[k / 4][k % 4];
        if (c > t) {
          *found = static_cast<int>(y0 + k);
          break;
        }
      }
    }
    base += total;
    if (base > t) break;   // uniform: every thread holds the same base
  }
  __syncthreads();
  return *found;
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void verify_kernel(VerifyArgs a) {
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int B = a.B, V = a.V;
  __shared__ uint64_t red[NW];
  __shared__ int sh_m, sh_found;
  const int64_t prow0 = static_cast<int64_t>(s) * (B + 1);
  const int64_t qrow0 = static_cast<int64_t>(s) * B;
  if (tid < 64) {
    int m = B;
    bool bad = false;
    for (int j0 = 0; j0 < B; j0 += 64) {
      const int j = j0 + lane;
      bool rej = false;
      if (j < B) {
        const int x = a.draft[qrow0 + j];
        if (x < 0 || x >= V) {
          bad = true;
        } else {
          const double u = static_cast<double>(a.words[prow0 + j] >> 8) * 0x1p-24;
          const double pj = a.p[(prow0 + j) * V + x];
          const double qj = a.q[(qrow0 + j) * V + x];
          rej = !(u * qj < pj);
        }
      }
      const unsigned long long mask = __ballot(rej);
      if (mask && m == B) m = j0 + __ffsll(static_cast<long long>(mask)) - 1;
    }
    bad = __any(bad);
    if (lane == 0) sh_m = bad ? -1 : m;
  }
  __syncthreads();
  const int m = sh_m;
  int32_t* bits = a.accept_bits + qrow0;
  for (int j = tid; j < B; j += 64 * NW) bits[j] = j < m ? 1 : 0;
  if (m < 0) {
    if (tid == 0) {
      a.accept_len[s] = 0;
      a.next_tok[s] = -1;
      set_status(a.status, CO_ERR_TOKEN);
    }
    return;
  }
  const float* p = a.p + (prow0 + m) * V;
  const float* q = m < B ? a.q + (qrow0 + m) * V : nullptr;
  const int R = wave_tokens<NW>(V);
  uint64_t W = row_total<NW>(p, q, V, R, red);
  if (W == 0 && q) {
    q = nullptr;
    W = row_total<NW>(p, q, V, R, red);
  }
  int next = -1;
  if (W) {
    const uint64_t u = a.words[prow0 + B];
    const uint64_t t = u * (W >> 32) + ((u * (W & 0xFFFFFFFFull)) >> 32);   // floor(u W / 2^32)
    next = row_find<NW>(p, q, V, R, t, red, &sh_found);
  }
  if (tid == 0) {
    a.accept_len[s] = m;
    a.next_tok[s] = next;
  }
}

}  // namespace

hipError_t launch_verify(const VerifyArgs& a, hipStream_t stream) {
  if (a.S == 0) return hipSuccess;
  // Wavefronts of a sequence's workgroup.  A long row wants sixteen, a short one is
  // done by eight; many sequences fill the chip by themselves, and what counts is
  // how many workgroups it holds at once (each a chain of barriers and two passes).
  // us with 2, 4, 8, 16 wavefronts: 32 x 128000 tokens 107, 45, 25, 20; 256 x 2000
  // 8, 8, 8, 11; 1024 x 1000 8, 8, 11, 23; 1024 x 32000 52, 43, 39, 49; 4096 x 1000
  // 14, 22, 41, 94; 4096 x 32000 193, 159, 150, 199.  (Four wavefronts also keep
  // S * threads within a launch's limit where sixteen would not.)  Short rows of still
  // more sequences take one: with 1 and 2 wavefronts 4096 x 16 8.5, 11.7; 4096 x 1000
  // 11, 15; 30000 x 100 43, 77; but 2048 x 1000 8.6, 8.4 and 8192 x 2000 41, 40.
  int nw = a.S <= 512 ? 8 : (a.S <= 1024 ? 4 : 2);
  if (a.V > 16384 && nw < 8) nw *= 2;
  if (a.V > 49152 && a.S <= 512) nw = 16;
  if (a.V <= 1024 && a.S > 2048) nw = 1;
  if (nw == 16) hipLaunchKernelGGL(verify_kernel<16>, dim3(a.S), dim3(1024), 0, stream, a);
  else if (nw == 8) hipLaunchKernelGGL(verify_kernel<8>, dim3(a.S), dim3(512), 0, stream, a);
  else if (nw == 4) hipLaunchKernelGGL(verify_kernel<4>, dim3(a.S), dim3(256), 0, stream, a);
  else if (nw == 2) hipLaunchKernelGGL(verify_kernel<2>, dim3(a.S), dim3(128), 0, stream, a);
  else hipLaunchKernelGGL(verify_kernel<1>, dim3(a.S), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace co

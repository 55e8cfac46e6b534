// Sign packing (Sec. 3.1, Eq. uv_sign) into LB layout v1, plus a zero-fill
// kernel for workspaces.
//
// Bit t of a word is set iff the element at reduction index 32 kb + t is
// negative (sign -1; +0, -0 and NaN give +1, NaNs are counted).  The source is
// read once and 32x less is written, so the call is the latency of its loads:
// both kernels have many independent loads per thread, with consecutive lanes
// on consecutive addresses.  One element at a time, and for role U each lane on
// a row of its own, took 10.6 us for either orientation of a 11008 x 128 fp32
// factor (5.6 MB); now 3.4 us (role U) and 4.2 us (role V), 2-3 us of it launch.
//   role V  (the reduction index runs down the rows): a thread builds one word,
//           32 loads a row apart, lanes over the latent columns;
//   role U  (it runs along a row): a wave takes 16 rows x 64 latents, a load a
//           row; the compare's lane mask is that row's two words.  Narrow
//           rows would leave most lanes idle: 64 rows as one stream of elements.
#include "device_common.h"

namespace lb {

namespace {

constexpr int kPackThreads = 256;
constexpr int kPackRows = 16;  // role U: rows per wave
// Role U, us for rows of r latents by 16 x 64 tiles against 64 rows a wave (bf16;
// fp32 alike): 11008 rows r = 1 3.2 / 2.4, r = 8 3.2 / 2.8, r = 16 3.2 / 3.7, r = 32
// 3.2 / 4.7; 262144 rows r = 1 10.1 / 2.5, r = 8 10.1 / 3.3, r = 16 9.9 / 4.7, r = 32 10.1 / 6.5
constexpr int kNarrow = 8;                // rows of at most this: 64 a wave
constexpr int kNarrowMany = 32;           // the same from kNarrowRows rows
constexpr int kNarrowRows = 1 << 17;

// A factor has fewer than 2^31 elements (the call checks), so the indices of its
// elements and the counts of words and of 16 x 64 tiles fit 32 bits unsigned; divides
// and products in 64 bits cost about 0.5 us a call (the eight packs of a 7B gate training
// step: 264.5 -> 260.0 us).

// word kb of output row o: a full word, or the tail plane's 16- or 32-bit entry
__device__ __forceinline__ void put_word(uint32_t* dst, int kb, int o, int nb, int w, int n_out, uint32_t word) {
  const int64_t n_full = static_cast<int64_t>(nb) * n_out;
  if (kb < nb)
    dst[static_cast<int64_t>(kb) * n_out + o] = word;
  else if (w <= 16)
    reinterpret_cast<uint16_t*>(dst + n_full)[o] = static_cast<uint16_t>(word);
  else
    dst[n_full + o] = word;
}

template <int DT>
__global__ void __launch_bounds__(kPackThreads) pack_v_kernel(const void* __restrict__ src, int rows, int r,
                                                              uint32_t* __restrict__ dst, int32_t* nan_count) {
  const int nb = rows >> 5, w = rows & 31;
  const uint32_t ur = r;
  const uint32_t item = blockIdx.x * kPackThreads + threadIdx.x;
  const uint32_t ukb = item / ur, uo = item - ukb * ur;
  if (ukb >= static_cast<uint32_t>(nb + (w != 0))) return;
  const int kb = static_cast<int>(ukb), o = static_cast<int>(uo);
  const int width = kb < nb ? 32 : w;
  const uint32_t base = 32u * ukb * ur + uo;
  uint32_t e[32];
#pragma unroll
  for (int t = 0; t < 32; ++t) e[t] = ld_bits<DT>(src, t < width ? base + t * ur : base);
  uint32_t word = 0;
  int nan = 0;
#pragma unroll
  for (int t = 0; t < 32; ++t) {
    const float v = bits_to_f32<DT>(e[t]);
    const bool in = t < width;
    word |= static_cast<uint32_t>(in && v < 0.0f) << t;
    nan += in && v != v;
  }
  put_word(dst, kb, o, nb, w, r, word);
  if (nan_count && nan) atomicAdd(nan_count, nan);
}

template <int DT>
__global__ void __launch_bounds__(kPackThreads) pack_u_kernel(const void* __restrict__ src, int rows, int r,
                                                              uint32_t* __restrict__ dst, int32_t* nan_count) {
  const int nb = r >> 5, w = r & 31, nkb = nb + (w != 0);
  const int lane = threadIdx.x & 63;
  const uint32_t nch = (nkb + 1) >> 1;  // 64-latent chunks
  const uint32_t unit = blockIdx.x * (kPackThreads / 64) + (threadIdx.x >> 6);
  const uint32_t ou = unit / nch * kPackRows;
  if (ou >= static_cast<uint32_t>(rows)) return;  // whole waves leave together
  const int o0 = static_cast<int>(ou), c = static_cast<int>(unit % nch);
  const int nrow = min(kPackRows, rows - o0);
  const uint32_t k = 64u * c + lane;
  const uint32_t ur = r;
  uint32_t e[kPackRows];
#pragma unroll
  for (int i = 0; i < kPackRows; ++i)
    e[i] = ld_bits<DT>(src, i < nrow && k < ur ? (ou + i) * ur + k : 0u);
  // lane 16 j + i: word 2 c + j of row o0 + i
  uint32_t word = 0;
  int nan = 0;
#pragma unroll
  for (int i = 0; i < kPackRows; ++i) {
    const float v = bits_to_f32<DT>(e[i]);
    const uint64_t m = __ballot(k < ur && v < 0.0f);
    if ((lane & 15) == i) word = static_cast<uint32_t>(lane & 16 ? m >> 32 : m);
    nan += i < nrow && k < ur && v != v;
  }
  const int kb = 2 * c + (lane >> 4), i = lane & 15;
  if (lane < 32 && i < nrow && kb < nkb) put_word(dst, kb, o0 + i, nb, w, rows, word);
  if (nan_count && nan) atomicAdd(nan_count, nan);
}

// r <= N (at most 32), so a row is one word or tail entry: a wave takes 64 rows,
// whose 64 r elements are read 64 consecutive ones at a time; the compare's r lane
// masks are 64 r consecutive bits, of which lane l takes those from l r on.
template <int DT, int N>
__global__ void __launch_bounds__(kPackThreads) pack_u_narrow_kernel(const void* __restrict__ src, int rows, int r,
                                                                     uint32_t* __restrict__ dst, int32_t* nan_count) {
  const int lane = threadIdx.x & 63;
  const int64_t o0 = (blockIdx.x * static_cast<int64_t>(kPackThreads / 64) + (threadIdx.x >> 6)) * 64;
  if (o0 >= rows) return;  // whole waves leave together
  const int nrow = static_cast<int>(min(static_cast<int64_t>(64), rows - o0));
  uint32_t e[N];
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < r) e[i] = ld_bits<DT>(src, o0 * r + (64 * i + lane < nrow * r ? 64 * i + lane : 0));
  uint64_t mask = 0;  // lane i: of elements 64 i .. 64 i + 63
  int nan = 0;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < r) {
      const float v = bits_to_f32<DT>(e[i]);
      const bool in = 64 * i + lane < nrow * r;
      const uint64_t m = __ballot(in && v < 0.0f);
      if (lane == i) mask = m;
      nan += in && v != v;
    }
  const int w = (lane * r) >> 6, sh = (lane * r) & 63;
  uint64_t bits = static_cast<uint64_t>(__shfl(static_cast<unsigned long long>(mask), w)) >> sh;
  const uint64_t next = __shfl(static_cast<unsigned long long>(mask), (w + 1) & 63);
  if (sh + r > 64) bits |= next << (64 - sh);
  const uint32_t word = static_cast<uint32_t>(bits & ((uint64_t(1) << r) - 1));
  if (lane < nrow) {
    if (r <= 16)
      reinterpret_cast<uint16_t*>(dst)[o0 + lane] = static_cast<uint16_t>(word);
    else
      dst[o0 + lane] = word;
  }
  if (nan_count && nan) atomicAdd(nan_count, nan);
}

template <int DT>
void launch_pack_t(const void* src, int rows, int r, int role, uint32_t* dst, int32_t* nan_count, hipStream_t stream) {
  if (role == LB_ROLE_U && (r <= kNarrow || (r <= kNarrowMany && rows >= kNarrowRows))) {
    const int64_t waves = (int64_t(rows) + 63) / 64, per = kPackThreads / 64;
    const dim3 grid(static_cast<uint32_t>((waves + per - 1) / per));
    if (r <= kNarrow)
      hipLaunchKernelGGL((pack_u_narrow_kernel<DT, kNarrow>), grid, dim3(kPackThreads), 0, stream, src, rows, r, dst,
                         nan_count);
    else
      hipLaunchKernelGGL((pack_u_narrow_kernel<DT, kNarrowMany>), grid, dim3(kPackThreads), 0, stream, src, rows, r, dst,
                         nan_count);
  } else if (role == LB_ROLE_U) {
    const int64_t waves = (int64_t(rows) + kPackRows - 1) / kPackRows * ((int64_t(r) + 63) / 64);
    const int64_t per = kPackThreads / 64;
    hipLaunchKernelGGL((pack_u_kernel<DT>), dim3(static_cast<uint32_t>((waves + per - 1) / per)), dim3(kPackThreads),
                       0, stream, src, rows, r, dst, nan_count);
  } else {
    const int64_t items = (int64_t(rows) + 31) / 32 * r;
    hipLaunchKernelGGL((pack_v_kernel<DT>), dim3(static_cast<uint32_t>((items + kPackThreads - 1) / kPackThreads)),
                       dim3(kPackThreads), 0, stream, src, rows, r, dst, nan_count);
  }
}

// Zero n_words 32-bit words, then one trailing 16-bit half-word if `half_tail`.
__global__ void __launch_bounds__(256) fill_zero_kernel(uint32_t* __restrict__ p, int64_t n_words, int half_tail) {
  const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  for (int64_t i = i0; i < n_words; i += static_cast<int64_t>(gridDim.x) * blockDim.x) p[i] = 0u;
  if (half_tail && i0 == 0) reinterpret_cast<uint16_t*>(p + n_words)[0] = 0;
}

__global__ void __launch_bounds__(256) zero_elems_kernel(void* __restrict__ p, int64_t n, int dt) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    store_from_f32(p, i, dt, 0.0f);
}

}  // namespace

hipError_t launch_zero_elems(void* p, int64_t n, int dt, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  const int grid = static_cast<int>(blocks < 8192 ? blocks : 8192);
  hipLaunchKernelGGL(zero_elems_kernel, dim3(grid), dim3(256), 0, stream, p, n, dt);
  return hipGetLastError();
}

hipError_t launch_pack(const void* src, int dt, int rows, int r, int role, void* dst, int32_t* nan_count,
                       hipStream_t stream) {
  if (rows == 0 || r == 0) return hipSuccess;
  uint32_t* d = static_cast<uint32_t*>(dst);
  switch (dt) {
    case kDtF32: launch_pack_t<kDtF32>(src, rows, r, role, d, nan_count, stream); break;
    case kDtF16: launch_pack_t<kDtF16>(src, rows, r, role, d, nan_count, stream); break;
    default: launch_pack_t<kDtBF16>(src, rows, r, role, d, nan_count, stream); break;
  }
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream) {
  // bytes must be a multiple of 2 and p 4-byte aligned
  const int64_t n = static_cast<int64_t>(bytes / 4);
  const int half_tail = (bytes % 4) != 0;
  if (n == 0 && !half_tail) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  const int grid = static_cast<int>(blocks < 1 ? 1 : (blocks < 8192 ? blocks : 8192));
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, stream, static_cast<uint32_t*>(p), n, half_tail);
  return hipGetLastError();
}

namespace {
__global__ void take_status_kernel(uint32_t* ctrl, int32_t* out) {
  const uint32_t v = __hip_atomic_exchange(ctrl + kCtrlError, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *out = static_cast<int32_t>(v);
}
}  // namespace

hipError_t launch_take_status(uint32_t* ctrl, int32_t* out, hipStream_t stream) {
  hipLaunchKernelGGL(take_status_kernel, dim3(1), dim3(1), 0, stream, ctrl, out);
  return hipGetLastError();
}

}  // namespace lb

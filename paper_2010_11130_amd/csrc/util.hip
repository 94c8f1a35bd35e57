// Device utilities: exclusive prefix sums used to turn per-row counts into
// CSR offsets.
#include <cstring>

#include "system.h"

namespace ah {

// Exclusive prefix sums in at most two launches: SCAN_PER values per thread, a
// tile per workgroup.  Up to one large tile a single workgroup does it all;
// beyond, the tiles' sums come first and every workgroup of the second launch
// adds up the sums before its own (at most 1024 of them with small tiles; large
// ones above that).  The setup is a chain of small dependent launches, so their
// number is what a scan costs: a tile pass with recursive scans of the sums, an
// addition and a total took two to five launches each (setup of 342,528 rows,
// nine levels: 2790 us with those and a copy per value read back, 2536 with these
// and polled reads).
constexpr int SCAN_PER = 16;
constexpr int SCAN_ONE = 1024 * SCAN_PER;
constexpr int SCAN_TILE = 256 * SCAN_PER;

// Sum over the workgroup's values before thread t's x, and of all of them.
template <int T>
__device__ inline int64_t block_prefix(int64_t x, int64_t* red, int64_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int64_t inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t u = __shfl_up(inc, o, 64);
    inc += lane >= o ? u : 0;
  }
  if (lane == 63) red[wv] = inc;
  __syncthreads();
  int64_t before = inc - x, all = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const int64_t r = red[w];
    before += w < wv ? r : 0;
    all += r;
  }
  *total = all;
  return before;
}

template <class T, int NT>
__global__ __launch_bounds__(NT) void k_scan_sums(const T* __restrict__ in, int64_t n, int64_t* __restrict__ sums) {
  __shared__ int64_t red[NT / 64];
  const int64_t base = (int64_t)blockIdx.x * (NT * SCAN_PER) + threadIdx.x;
  int64_t x = 0;
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    const int64_t i = base + (int64_t)q * NT;
    x += i < n ? (int64_t)in[i] : 0;
  }
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    sums[blockIdx.x] = t;
  }
}

// The tile's prefix sums; sums null: a single tile.
template <class T, int NT>
__global__ __launch_bounds__(NT) void k_scan_out(const T* __restrict__ in, int64_t n,
                                                 const int64_t* __restrict__ sums, int64_t* __restrict__ out) {
  __shared__ int64_t red[2][NT / 64];
  int64_t carry = 0;
  if (sums) {
    int64_t x = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += NT) x += sums[b];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = x;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) carry += red[0][w];
  }
  const int64_t base = ((int64_t)blockIdx.x * NT + threadIdx.x) * SCAN_PER;
  int64_t v[SCAN_PER], tot = 0;
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    v[q] = base + q < n ? (int64_t)in[base + q] : 0;
    tot += v[q];
  }
  int64_t all = 0;
  int64_t run = carry + block_prefix<NT>(tot, red[1], &all);
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    if (base + q < n) out[base + q] = run;
    run += v[q];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = carry + all;
}

template <class T>
static ah_status scan_impl(const T* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp) {
  if (n <= SCAN_ONE) {
    hipLaunchKernelGGL((k_scan_out<T, 1024>), dim3(1), dim3(1024), 0, st, in, n, (const int64_t*)nullptr, out);
    AH_LAUNCHED();
    return AH_OK;
  }
  const bool large = n > 1024 * (int64_t)SCAN_TILE;
  const int64_t nb = cdiv(n, large ? SCAN_ONE : SCAN_TILE);
  int64_t* sums = nullptr;
  AH_TRY(tmp.get(&sums, nb));
  if (large) {
    hipLaunchKernelGGL((k_scan_sums<T, 1024>), dim3((unsigned)nb), dim3(1024), 0, st, in, n, sums);
    hipLaunchKernelGGL((k_scan_out<T, 1024>), dim3((unsigned)nb), dim3(1024), 0, st, in, n, sums, out);
  } else {
    hipLaunchKernelGGL((k_scan_sums<T, 256>), dim3((unsigned)nb), dim3(256), 0, st, in, n, sums);
    hipLaunchKernelGGL((k_scan_out<T, 256>), dim3((unsigned)nb), dim3(256), 0, st, in, n, sums, out);
  }
  AH_LAUNCHED();
  return AH_OK;
}

ah_status scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp) {
  return scan_impl<int64_t>(in, out, n, st, tmp);
}

ah_status scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp) {
  return scan_impl<int32_t>(in, out, n, st, tmp);
}

// Copies the words of up to READ_MAX device values into pinned host memory,
// then seq into the flag that the host polls.
constexpr int READ_MAX = 6;
constexpr int READ_WORDS = 16;
struct ReadArgs {
  const uint32_t* src[READ_MAX];
  int words[READ_MAX];
};

__global__ __launch_bounds__(128) void k_read(ReadArgs a, uint32_t* host, unsigned long long* flag,
                                              unsigned long long seq) {
  const int v = threadIdx.x / READ_WORDS, w = threadIdx.x % READ_WORDS;
  if (v < READ_MAX && w < a.words[v]) host[v * READ_WORDS + w] = a.src[v][w];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

ah_status poll_flag(const unsigned long long* flag, unsigned long long seq, hipStream_t st) {
  for (unsigned spin = 1; __atomic_load_n(flag, __ATOMIC_ACQUIRE) != seq; ++spin) {
    __builtin_ia32_pause();
    if (spin % 65536) continue;
    // a stream that has stopped will not set the flag any more
    const hipError_t e = hipStreamQuery(st);
    (void)hipGetLastError();   // "not ready" is no error of a later launch
    if (e == hipErrorNotReady || __atomic_load_n(flag, __ATOMIC_ACQUIRE) == seq) continue;
    set_error("%s", e == hipSuccess ? "device result missing" : hipGetErrorString(e));
    return AH_EHIP;
  }
  return AH_OK;
}

ah_status read_values(std::initializer_list<ReadItem> items, hipStream_t st) {
  // the last 64 doubles of the smallest pinned buffer: values, then the flag
  constexpr size_t AT = 8192 - 64;
  static_assert(READ_MAX * READ_WORDS * 4 + 8 <= 64 * 8, "values and flag");
  static thread_local unsigned long long seq = 0;
  double* pin = pinned_scratch(AT + 64);
  if (!pin) { set_error("pinned host allocation failed"); return AH_ENOMEM; }
  uint32_t* host = reinterpret_cast<uint32_t*>(pin + AT);
  unsigned long long* flag = reinterpret_cast<unsigned long long*>(pin + AT + 63);
  ReadArgs a{};
  int n = 0;
  for (const ReadItem& it : items) {
    if (n == READ_MAX || it.bytes % 4 || it.bytes > READ_WORDS * 4) {
      set_error("read_values: bad item");
      return AH_EINVAL;
    }
    a.src[n] = static_cast<const uint32_t*>(it.dev);
    a.words[n++] = (int)(it.bytes / 4);
  }
  __atomic_store_n(flag, 0ull, __ATOMIC_RELEASE);
  hipLaunchKernelGGL(k_read, dim3(1), dim3(128), 0, st, a, host, flag, ++seq);
  AH_LAUNCHED();
  AH_TRY(poll_flag(flag, seq, st));
  n = 0;
  for (const ReadItem& it : items) std::memcpy(it.host, host + READ_WORDS * n++, it.bytes);
  return AH_OK;
}

ah_status read_i64(const int64_t* d, int64_t* h, hipStream_t st) { return read_values({{d, h, sizeof(int64_t)}}, st); }

ah_status read_bytes(const void* d, void* h, size_t bytes, hipStream_t st) {
  return read_values({{d, h, bytes}}, st);
}

}  // namespace ah

// Device utilities: exclusive prefix sums used to turn per-row counts into
// CSR offsets.
#include <cstring>

#include "system.h"

namespace ah {

// The words of up to READ_MAX device values for pinned host memory, and then seq
// for the flag that the host polls; flag null: nothing.
constexpr int READ_MAX = 6;
constexpr int READ_WORDS = 16;
struct ReadArgs {
  const uint32_t* src[READ_MAX];
  int words[READ_MAX];
  uint32_t* host;
  unsigned long long* flag;
  unsigned long long seq;
};

// The copy, by the workgroup's first wave: one wave's stores and one fence (a
// fence by each of 16 waves took 8 us).
__device__ inline void read_out(const ReadArgs& a) {
  if (threadIdx.x >= 64) return;
  for (int x = threadIdx.x; x < READ_MAX * READ_WORDS; x += 64) {
    const int v = x / READ_WORDS, w = x % READ_WORDS;
    if (w < a.words[v]) a.host[x] = a.src[v][w];
  }
  __threadfence_system();
  if (threadIdx.x == 0) __hip_atomic_store(a.flag, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Exclusive prefix sums in at most two launches: SCAN_PER values per thread, a
// tile per workgroup.  Up to one large tile a single workgroup does it all;
// beyond, the tiles' sums come first and every workgroup of the second launch
// adds up the sums before its own (at most 1024 of them with small tiles; large
// ones above that).  The setup is a chain of small dependent launches, so their
// number is what a scan costs: a tile pass with recursive scans of the sums, an
// addition and a total took two to five launches each (setup of 342,528 rows,
// nine levels: 2790 us with those and a copy per value read back, 2536 with these
// and polled reads).
// A tile is CH chunks of four neighbouring values per thread, so a wave
// reads 1 KiB and writes 2 KiB in one piece each time; 16 values in a row per
// thread made every store touch 64 lines (14,912 values in one workgroup: 16 us,
// 8 now)
// (one chunk up to 4096 values in one workgroup: a shorter chain).
constexpr int SCAN_CH = 4;
constexpr int SCAN_PER = 4 * SCAN_CH;
constexpr int SCAN_ONE = 1024 * SCAN_PER;
constexpr int SCAN_TILE = 256 * SCAN_PER;

// in[base .. base + 3], zero from n on; vec: 16-byte aligned arrays.
template <class T>
__device__ inline void scan_load(const T* __restrict__ in, int64_t base, int64_t n, int vec, T (&v)[4]) {
  typedef int I4 __attribute__((ext_vector_type(4)));
  typedef long L2 __attribute__((ext_vector_type(2)));
  if (vec && base + 4 <= n) {
    if constexpr (sizeof(T) == 4) {
      const I4 x = *reinterpret_cast<const I4*>(in + base);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
      const L2 x = *reinterpret_cast<const L2*>(in + base), y = *reinterpret_cast<const L2*>(in + base + 2);
      v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = base + q < n ? in[base + q] : 0;
}

__device__ inline int64_t wave_sum(int64_t x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ inline int64_t wave_max(int64_t x) {
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t y = __shfl_xor(x, o, 64);
    x = y > x ? y : x;
  }
  return x;
}

// Sums of the tiles, then (from sums + gridDim.x) their largest values.
template <class T, int NT>
__global__ __launch_bounds__(NT) void k_scan_sums(const T* __restrict__ in, int64_t n, int vec,
                                                  int64_t* __restrict__ sums) {
  __shared__ int64_t red[2][NT / 64];
  const int64_t base = (int64_t)blockIdx.x * (NT * SCAN_PER) + threadIdx.x * 4;
  T v[SCAN_CH][4];
#pragma unroll
  for (int c = 0; c < SCAN_CH; ++c) scan_load(in, base + c * (NT * 4), n, vec, v[c]);
  int64_t x = 0, m = 0;
#pragma unroll
  for (int c = 0; c < SCAN_CH; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x += v[c][q];
      m = v[c][q] > m ? v[c][q] : m;
    }
  x = wave_sum(x);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = x;
    red[1][threadIdx.x >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NT / 64; ++w) {
      x += red[0][w];
      m = red[1][w] > m ? red[1][w] : m;
    }
    sums[blockIdx.x] = x;
    sums[gridDim.x + blockIdx.x] = m;
  }
}

// The tile's prefix sums; sums null: a single tile.  The last tile also writes
// the total to out[n] and, where vmax is given, the largest value (at least 0).
// zero (or null): n values cleared on the way.  A single tile can also hand
// values to the host when it is done, its own among them.
template <class T, int NT, int CH>
__global__ __launch_bounds__(NT) void k_scan_out(const T* __restrict__ in, int64_t n, int vec,
                                                 const int64_t* __restrict__ sums, int64_t* __restrict__ out,
                                                 int* __restrict__ vmax, int32_t* __restrict__ zero,
                                                 ReadArgs rd) {
  constexpr int W = NT / 64;
  __shared__ int64_t red[2][W], part[CH * W];
  typedef long L2 __attribute__((ext_vector_type(2)));
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const bool last = blockIdx.x == gridDim.x - 1;
  const int64_t base = (int64_t)blockIdx.x * (NT * 4 * CH) + t * 4;
  T v[CH][4];
#pragma unroll
  for (int c = 0; c < CH; ++c) scan_load(in, base + c * (NT * 4), n, vec, v[c]);
  int64_t before = 0, m = 0;
  if (sums) {
    for (int b = t; b < (int)blockIdx.x; b += NT) before += sums[b];
    if (last && vmax)
      for (int b = t; b < (int)gridDim.x; b += NT) m = sums[gridDim.x + b] > m ? sums[gridDim.x + b] : m;
  } else if (vmax) {
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) m = v[c][q] > m ? v[c][q] : m;
  }
  if (sums) before = wave_sum(before);
  if (vmax) m = wave_max(m);
  if (lane == 0) {
    red[0][w] = before;
    red[1][w] = m;
  }
  // inclusive sums over the lanes of each chunk
  int64_t own[CH], inc[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) own[c] = inc[c] = (int64_t)v[c][0] + v[c][1] + v[c][2] + v[c][3];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int64_t u = __shfl_up(inc[c], o, 64);
      inc[c] += lane >= o ? u : 0;
    }
  if (lane == 63)
#pragma unroll
    for (int c = 0; c < CH; ++c) part[c * W + w] = inc[c];
  __syncthreads();
  if (t < 64) {   // the first wave scans the waves' sums, chunk by chunk
    int64_t carry = 0;
    for (int k = 0; k < W; ++k) carry += red[0][k];
    const int64_t x = t < CH * W ? part[t] : 0;
    int64_t y = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t u = __shfl_up(y, o, 64);
      y += t >= o ? u : 0;
    }
    if (t < CH * W) part[t] = carry + y - x;
    if (last && t == 63) {
      out[n] = carry + y;
      if (vmax) {
        for (int k = 0; k < W; ++k) m = red[1][k] > m ? red[1][k] : m;
        *vmax = (int)m;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int64_t i = base + c * (NT * 4);
    const int64_t r0 = part[c * W + w] + inc[c] - own[c];
    const int64_t r1 = r0 + v[c][0], r2 = r1 + v[c][1], r3 = r2 + v[c][2];
    if (vec && i + 4 <= n) {
      *reinterpret_cast<L2*>(out + i) = L2{r0, r1};
      *reinterpret_cast<L2*>(out + i + 2) = L2{r2, r3};
    } else {
      if (i < n) out[i] = r0;
      if (i + 1 < n) out[i + 1] = r1;
      if (i + 2 < n) out[i + 2] = r2;
      if (i + 3 < n) out[i + 3] = r3;
    }
    if (zero) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i + q < n) zero[i + q] = 0;
    }
  }
  if (rd.flag) {
    __syncthreads();   // total and largest value, written by the first wave too
    read_out(rd);
  }
}

template <class T>
static ah_status scan_impl(const T* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp, int* vmax, int32_t* zero,
                           const ReadArgs& rd) {
  const int vec = (reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) % 16 == 0;
  if (n <= 4096) {
    hipLaunchKernelGGL((k_scan_out<T, 1024, 1>), dim3(1), dim3(1024), 0, st, in, n, vec, (const int64_t*)nullptr, out,
                       vmax, zero, rd);
    AH_LAUNCHED();
    return AH_OK;
  }
  if (n <= SCAN_ONE) {
    hipLaunchKernelGGL((k_scan_out<T, 1024, SCAN_CH>), dim3(1), dim3(1024), 0, st, in, n, vec, (const int64_t*)nullptr, out,
                       vmax, zero, rd);
    AH_LAUNCHED();
    return AH_OK;
  }
  const bool large = n > 1024 * (int64_t)SCAN_TILE;
  const int64_t nb = cdiv(n, large ? SCAN_ONE : SCAN_TILE);
  int64_t* sums = nullptr;
  AH_TRY(tmp.get(&sums, 2 * nb));
  if (large) {
    hipLaunchKernelGGL((k_scan_sums<T, 1024>), dim3((unsigned)nb), dim3(1024), 0, st, in, n, vec, sums);
    hipLaunchKernelGGL((k_scan_out<T, 1024, SCAN_CH>), dim3((unsigned)nb), dim3(1024), 0, st, in, n, vec, sums, out, vmax,
                       zero, rd);
  } else {
    hipLaunchKernelGGL((k_scan_sums<T, 256>), dim3((unsigned)nb), dim3(256), 0, st, in, n, vec, sums);
    hipLaunchKernelGGL((k_scan_out<T, 256, SCAN_CH>), dim3((unsigned)nb), dim3(256), 0, st, in, n, vec, sums, out, vmax,
                       zero, rd);
  }
  AH_LAUNCHED();
  return AH_OK;
}

ah_status scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp) {
  return scan_impl<int64_t>(in, out, n, st, tmp, nullptr, nullptr, ReadArgs{});
}

ah_status scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp, int* vmax) {
  return scan_impl<int32_t>(in, out, n, st, tmp, vmax, nullptr, ReadArgs{});
}

__global__ __launch_bounds__(64) void k_read(ReadArgs a) { read_out(a); }

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

// The kernel's arguments for the items, the thread's pinned buffer and the next
// number of its flag.
static ah_status read_args(std::initializer_list<ReadItem> items, ReadArgs* a) {
  // the last 64 doubles of the smallest pinned buffer: values, then the flag
  constexpr size_t AT = 8192 - 64;
  static_assert(READ_MAX * READ_WORDS * 4 + 8 <= 64 * 8, "values and flag");
  static thread_local unsigned long long seq = 0;
  double* pin = pinned_scratch(AT + 64);
  if (!pin) { set_error("pinned host allocation failed"); return AH_ENOMEM; }
  *a = ReadArgs{};
  a->host = reinterpret_cast<uint32_t*>(pin + AT);
  a->flag = reinterpret_cast<unsigned long long*>(pin + AT + 63);
  a->seq = ++seq;
  int n = 0;
  for (const ReadItem& it : items) {
    if (n == READ_MAX || it.bytes % 4 || it.bytes > READ_WORDS * 4) {
      set_error("read_values: bad item");
      return AH_EINVAL;
    }
    a->src[n] = static_cast<const uint32_t*>(it.dev);
    a->words[n++] = (int)(it.bytes / 4);
  }
  __atomic_store_n(a->flag, 0ull, __ATOMIC_RELEASE);
  return AH_OK;
}

static ah_status read_wait(std::initializer_list<ReadItem> items, const ReadArgs& a, hipStream_t st) {
  AH_TRY(poll_flag(a.flag, a.seq, st));
  int n = 0;
  for (const ReadItem& it : items) std::memcpy(it.host, a.host + READ_WORDS * n++, it.bytes);
  return AH_OK;
}

ah_status read_values(std::initializer_list<ReadItem> items, hipStream_t st) {
  ReadArgs a;
  AH_TRY(read_args(items, &a));
  hipLaunchKernelGGL(k_read, dim3(1), dim3(64), 0, st, a);
  AH_LAUNCHED();
  return read_wait(items, a, st);
}

ah_status scan_i32_read(const int32_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp, int* vmax,
                        int32_t* zero, std::initializer_list<ReadItem> items) {
  if (n > SCAN_ONE) {
    AH_TRY(scan_impl<int32_t>(in, out, n, st, tmp, vmax, zero, ReadArgs{}));
    return read_values(items, st);
  }
  ReadArgs a;
  AH_TRY(read_args(items, &a));
  AH_TRY(scan_impl<int32_t>(in, out, n, st, tmp, vmax, zero, a));
  return read_wait(items, a, st);
}

ah_status read_i64(const int64_t* d, int64_t* h, hipStream_t st) { return read_values({{d, h, sizeof(int64_t)}}, st); }

ah_status read_bytes(const void* d, void* h, size_t bytes, hipStream_t st) {
  return read_values({{d, h, bytes}}, st);
}

}  // namespace ah

// Data-movement and helper kernels of the SAR chain: the LDS-tiled corner
// turn, storage-format conversion and the per-pulse phasor table used by the
// autofocus phase correction.
#include "fft_device.hpp"
#include "internal.hpp"

namespace bfp {

// ------------------------------------------------------------ corner turn --
// out[c][r] = in[r][c].  A 256-thread workgroup moves a tile of 64 input rows
// by TC input columns: it is read row by row (coalesced), staged in LDS with
// one element of padding per row, and written row by row of the output.  Tiles
// are assigned row-major over the output so that consecutive workgroups write
// neighbouring output rows.  Each lane reads VL consecutive elements of an
// input row and writes VS consecutive elements of an output row, each width
// where that side's rows are whole, aligned chunks: a matrix with an odd
// number of rows is still read 16 bytes per lane.  With TC = 128 each input
// row segment is 512 bytes (4-byte elements), which measured 5% faster on
// 4096 x 4096 than 64 x 64 tiles (25.0 against 26.4 us) although the staging
// writes into LDS then meet 2-way bank conflicts; the reads out of LDS stay
// conflict-free at the padded stride (bank of tile[r][c] = r + c mod 64).
//
// VS = 1: an output row starts anywhere in a cache line, so a tile's segment
// shares its first and last lines with the neighbouring tiles of the row.
// Those lines are merged in L2 (plain stores) where both tiles run on one
// XCD: the tiles are dealt in runs of consecutive ones per XCD (workgroup w
// runs on XCD w mod 8).
//
// VL = 1: the segments read share lines too, so the loads are plain ones, and
// the tile is 64 columns wide: a wavefront still reads a whole segment, and at
// 128 the 32 loads per lane take twice as long as the writes.  4095 x 4095
// FP16: 31 us at TC = 128, 50 us with nontemporal loads as well, 22 us so.
// (With narrow writes alone, plain loads take 9.8 against 11.2 us for
// 1531 x 4096 FP16 out of the caches and 12.7 against 11.3 from HBM.)
template <class T, int VL, int VS, int TC>
__global__ void __launch_bounds__(256) transpose_kernel(const T *__restrict__ in, T *__restrict__ out,
                                                        int rows, int cols, int tiles) {
  typedef T vin __attribute__((ext_vector_type(VL)));
  typedef T vout __attribute__((ext_vector_type(VS)));
  constexpr int CH = TC / VL;   // chunks per tile row
  constexpr int RPI = 256 / CH; // tile rows per iteration
  constexpr int CHO = 64 / VS;  // chunks per output row of the tile
  constexpr int RPO = 256 / CHO;
  static_assert(256 % CH == 0 && 64 % RPI == 0 && TC % RPO == 0, "tile shape");
  __shared__ T tile[64][TC + 1];
  const int tiles_r = (rows + 63) / 64;
  int b = blockIdx.x;
  if constexpr (VS == 1) {
    const int q = tiles >> 3, rem = tiles & 7, x = b & 7;
    b = x * q + (x < rem ? x : rem) + (b >> 3);
  }
  const int tc = b / tiles_r;
  const int tr = b % tiles_r;
  const int r0 = tr * 64, c0 = tc * TC;
  const int ch = threadIdx.x % CH, rl = threadIdx.x / CH;
#pragma unroll
  for (int k = 0; k < 64 / RPI; ++k) {
    const int rr = rl + RPI * k;
    const int r = r0 + rr, c = c0 + VL * ch;
    if (r < rows && c < cols) {
      const vin *src = reinterpret_cast<const vin *>(in + (size_t)r * cols + c);
      vin x;
      if constexpr (VL == 1 || VS == 1) x = *src;
      else x = __builtin_nontemporal_load(src);
#pragma unroll
      for (int u = 0; u < VL; ++u) tile[rr][VL * ch + u] = x[u];
    }
  }
  __syncthreads();
  const int cho = threadIdx.x % CHO, ro = threadIdx.x / CHO;
#pragma unroll
  for (int k = 0; k < TC / RPO; ++k) {
    const int oc = ro + RPO * k;      // output row within the tile = input column
    const int orow = c0 + oc, ocol = r0 + VS * cho;
    if (orow < cols && ocol < rows) {
      vout x;
#pragma unroll
      for (int u = 0; u < VS; ++u) x[u] = tile[VS * cho + u][oc];
      vout *dst = reinterpret_cast<vout *>(out + (size_t)orow * rows + ocol);
      if constexpr (VS == 1) *dst = x;
      else __builtin_nontemporal_store(x, dst);
    }
  }
}

template <class T, int V, int TC>
static hipError_t launch_transpose_of(const void *in, void *out, int rows, int cols, hipStream_t s) {
  const bool wide_in = cols % V == 0 && (uintptr_t)in % (V * sizeof(T)) == 0;
  const int width = wide_in ? TC : 64;
  const long long tiles = (long long)((rows + 63) / 64) * ((cols + width - 1) / width);
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  const bool wide_out = rows % V == 0 && (uintptr_t)out % (V * sizeof(T)) == 0;
  const T *src = static_cast<const T *>(in);
  T *dst = static_cast<T *>(out);
  const dim3 grid((unsigned)tiles), block(256);
  if (wide_in && wide_out)
    hipLaunchKernelGGL((transpose_kernel<T, V, V, TC>), grid, block, 0, s, src, dst, rows, cols, (int)tiles);
  else if (wide_in)
    hipLaunchKernelGGL((transpose_kernel<T, V, 1, TC>), grid, block, 0, s, src, dst, rows, cols, (int)tiles);
  else if (wide_out)
    hipLaunchKernelGGL((transpose_kernel<T, 1, V, 64>), grid, block, 0, s, src, dst, rows, cols, (int)tiles);
  else
    hipLaunchKernelGGL((transpose_kernel<T, 1, 1, 64>), grid, block, 0, s, src, dst, rows, cols, (int)tiles);
  return hipGetLastError();
}

hipError_t launch_transpose(const void *in, void *out, int rows, int cols, int bytes,
                            hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  switch (bytes) {
    case 2: return launch_transpose_of<uint16_t, 4, 128>(in, out, rows, cols, s);
    case 4: return launch_transpose_of<uint32_t, 4, 128>(in, out, rows, cols, s);
    case 8: return launch_transpose_of<uint64_t, 2, 64>(in, out, rows, cols, s);
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------- convert ----
// Storage of one format: the complex element as stored, and its exact FP32
// value.  FP32 -> FP16 rounds once (RNE); FP16/FP8 inputs are exact in FP32,
// so every conversion is a single correct rounding of the input value.
template <int FMT> struct Format;
template <> struct Format<0> {
  typedef c32 E;
  static __device__ __forceinline__ c32 get(E e) { return e; }
  static __device__ __forceinline__ E put(c32 v) { return v; }
};
template <> struct Format<1> {
  typedef h2 E;
  static __device__ __forceinline__ c32 get(E e) { return h2_to_c32(e); }
  static __device__ __forceinline__ E put(c32 v) { return c32_to_h2(v); }
};
template <int MANT> struct FormatFp8 {
  typedef uint16_t E;
  static __device__ __forceinline__ c32 get(E e) { return Fp8Codec<MANT>::decode2(e); }
  static __device__ __forceinline__ E put(c32 v) { return (E)Fp8Codec<MANT>::encode2(v.x, v.y); }
};
template <> struct Format<2> : FormatFp8<3> {};
template <> struct Format<3> : FormatFp8<2> {};

// V consecutive elements as one access
template <class E, int V>
struct alignas(V * sizeof(E)) Chunk {
  E e[V];
};

// Bound by HBM: the formats are compile-time, a lane moves V = 2 elements per
// access where both pointers are aligned for it (16 bytes of FP32, 8 of
// FP16) and keeps kConvertUnroll loads in flight; the run-time format switch
// per element that this replaces took 15.4 us for 1531 x 4096 FP32 -> FP16
// (75 MB).
constexpr int kConvertUnroll = 4;

template <int IN, int OUT, int V>
__global__ void __launch_bounds__(256) convert_kernel(const void *in, void *out, long long count) {
  typedef Format<IN> I;
  typedef Format<OUT> O;
  typedef Chunk<typename I::E, V> CI;
  typedef Chunk<typename O::E, V> CO;
  const CI *src = static_cast<const CI *>(in);
  CO *dst = static_cast<CO *>(out);
  const long long chunks = count / V;
  const long long step = 256LL * kConvertUnroll;
  for (long long base = blockIdx.x * step + threadIdx.x; base < chunks; base += gridDim.x * step) {
    CI x[kConvertUnroll];
#pragma unroll
    for (int u = 0; u < kConvertUnroll; ++u)
      if (base + 256 * u < chunks) x[u] = src[base + 256 * u];
#pragma unroll
    for (int u = 0; u < kConvertUnroll; ++u)
      if (base + 256 * u < chunks) {
        CO y;
#pragma unroll
        for (int v = 0; v < V; ++v) y.e[v] = O::put(I::get(x[u].e[v]));
        dst[base + 256 * u] = y;
      }
  }
  if constexpr (V > 1) {  // the elements after the last whole chunk
    const long long i = chunks * V + threadIdx.x;
    if (blockIdx.x == 0 && i < count)
      static_cast<typename O::E *>(out)[i] = O::put(I::get(static_cast<const typename I::E *>(in)[i]));
  }
}

template <int IN, int OUT>
static void launch_convert_of(const void *in, void *out, long long count, hipStream_t s) {
  const bool wide = (uintptr_t)in % (2 * sizeof(typename Format<IN>::E)) == 0 &&
                    (uintptr_t)out % (2 * sizeof(typename Format<OUT>::E)) == 0;
  const long long per = 256LL * kConvertUnroll * (wide ? 2 : 1);
  long long blocks = (count + per - 1) / per;
  if (blocks > 65536) blocks = 65536;
  const dim3 grid((unsigned)blocks), block(256);
  if (wide) hipLaunchKernelGGL((convert_kernel<IN, OUT, 2>), grid, block, 0, s, in, out, count);
  else hipLaunchKernelGGL((convert_kernel<IN, OUT, 1>), grid, block, 0, s, in, out, count);
}

template <int IN>
static hipError_t launch_convert_from(const void *in, void *out, int out_fmt, long long count, hipStream_t s) {
  switch (out_fmt) {
    case 0: launch_convert_of<IN, 0>(in, out, count, s); break;
    case 1: launch_convert_of<IN, 1>(in, out, count, s); break;
    case 2: launch_convert_of<IN, 2>(in, out, count, s); break;
    case 3: launch_convert_of<IN, 3>(in, out, count, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_convert(const void *in, int in_fmt, void *out, int out_fmt, long long count,
                          hipStream_t s) {
  if (count <= 0) return hipSuccess;
  switch (in_fmt) {
    case 0: return launch_convert_from<0>(in, out, out_fmt, count, s);
    case 1: return launch_convert_from<1>(in, out, out_fmt, count, s);
    case 2: return launch_convert_from<2>(in, out, out_fmt, count, s);
    case 3: return launch_convert_from<3>(in, out, out_fmt, count, s);
  }
  return hipErrorInvalidValue;
}

// -------------------------------------------------------------- phasor ----
// p[m] = exp(+/- i phase[m]) for the per-pulse phase correction; evaluated in
// FP64 from the FP32 radians and rounded once to FP32.
__global__ void __launch_bounds__(256) phasor_kernel(const float *__restrict__ phase,
                                                     c32 *__restrict__ p, int n, int negate) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    double s, c;
    sincos((double)phase[i], &s, &c);
    p[i] = c32{(float)c, (float)(negate ? -s : s)};
  }
}

hipError_t launch_phasor(const float *phase, void *phasor, int n, int negate, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(phasor_kernel, dim3((n + 255) / 256), dim3(256), 0, s, phase,
                     static_cast<c32 *>(phasor), n, negate);
  return hipGetLastError();
}

// ------------------------------------------------------------- copy ------
// Plain streaming copy: the reference for achievable HBM bandwidth and for
// calibrating memory counters.  Each thread keeps four 16-byte loads in
// flight (the workgroup moves 16 KiB per trip, lanes contiguous within each
// 4 KiB slice); the tail that is not a whole 16 KiB chunk is copied by a
// second, element-wise loop.
constexpr int kCopyUnroll = 4;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) copy_kernel(const u32x4 *__restrict__ in,
                                                   u32x4 *__restrict__ out, long long n16) {
  const long long chunk = 256LL * kCopyUnroll;
  const long long chunks = n16 / chunk;
  for (long long c = blockIdx.x; c < chunks; c += gridDim.x) {
    const u32x4 *src = in + c * chunk + threadIdx.x;
    u32x4 *dst = out + c * chunk + threadIdx.x;
    u32x4 v[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) v[u] = __builtin_nontemporal_load(src + 256 * u);
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) __builtin_nontemporal_store(v[u], dst + 256 * u);
  }
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = chunks * chunk + (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += stride)
    out[i] = in[i];
}

hipError_t launch_copy(const void *in, void *out, long long bytes, hipStream_t s) {
  const long long n16 = bytes / 16;
  if (n16 <= 0) return hipSuccess;
  long long blocks = (n16 + 256LL * kCopyUnroll - 1) / (256LL * kCopyUnroll);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const u32x4 *>(in), static_cast<u32x4 *>(out), n16);
  return hipGetLastError();
}

}  // namespace bfp

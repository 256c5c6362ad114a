// MX-FP8 quantisation of bf16 rows (the storage of a quantised Q K^T; the Conclusion,
// Section 5, lists quantisation among the methods the rule combines with), optionally of rows minus
// a float32 shift vector (key smoothing), and the per-head mean key that serves as that
// shift.
//
// Every run of 32 consecutive values of a row is one block: it shares the power-of-two
// scale 2^E with E = floor(log2(max |x|)) - 8, stored as the E8M0 code E + 127 (0 for an
// all-zero block), and each value becomes the FP8 E4M3 number nearest to x / 2^E -- ties
// to the even code, magnitudes above 448 saturating to 448.
//
// Four lanes share a block, eight values (one 16-byte load, one 8-byte store) each, so
// every load and store of a wave covers consecutive bytes; a thread keeps kChunks loads
// in flight.  The codes come from the hardware's pair conversion.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "quant_launch.h"

namespace dsattn {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kChunks = 4;               // 8-value chunks per thread
constexpr int kChunkValues = 8;

// E4M3 codes of four floats (byte i from y[i]), rounded to nearest with ties to the even
// code, magnitudes above 448 and NaN to 448 (0x7e), with the signs in bits 7, 15, 23 and 31 of
// `signs` except where the value rounds to zero: +0 (bit 7 of `nz` is set where a byte of the
// magnitudes' codes is not zero).
__device__ __forceinline__ uint32_t e4m3_codes(const float* y, uint32_t signs) {
  float c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) c[i] = fminf(fabsf(y[i]), 448.0f);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w, true);
  const uint32_t low = (uint32_t)w;
  const uint32_t nz = low + 0x7f7f7f7fu;
  return low | (signs & nz & 0x80808080u);
}

// Maximum over the four lanes of an aligned quad.
__device__ __forceinline__ uint32_t quad_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true));  // lane ^ 1
  x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true));  // lane ^ 2
  return x;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// One 8-value chunk: the block's scale code (the same in its four lanes) and this lane's
// eight codes.  `sh` holds the shift of the chunk's columns (SHIFT only): every value first
// has it subtracted (rounded to nearest float32).
template <bool SHIFT>
__device__ __forceinline__ void quantize_chunk(const u32x4& w, const float (&sh)[kChunkValues],
                                               u32x2& out, uint32_t& scode) {
  float x[kChunkValues];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] = bf16_lo(w[j]);
    x[2 * j + 1] = bf16_hi(w[j]);
  }
  // Bit pattern of max |x| over the block's numbers: magnitudes order as integers, and a NaN
  // counts as zero.
  uint32_t amax;
  if constexpr (SHIFT) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < kChunkValues; ++i) {
      x[i] -= sh[i];
      m = fmaxf(m, fabsf(x[i]));
    }
    amax = __float_as_uint(m);
  } else {
    // Plus 0x7f, magnitudes up to infinity's 0x7f80 stay positive 16-bit integers and a NaN's
    // turn negative, below zero's.
    i16x2 m{0x7f, 0x7f};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      m = __builtin_elementwise_max(
          m, __builtin_bit_cast(i16x2, (w[j] & 0x7fff7fffu) + 0x007f007fu));
    amax = (uint32_t)(max(m[0], m[1]) - 0x7f) << 16;
  }
  amax = quad_max(amax);
  // floor(log2 amax) - 8 + 127 is the biased exponent minus 8; zero and tiny blocks (and
  // subnormal maxima, whose biased exponent is 0) clamp to code 0.  Blocks with an infinity
  // take the scale 2^-9.
  scode = amax >= 0x7f800000u ? 118u : (uint32_t)max(0, (int)(amax >> 23) - 8);
  const float inv = __uint_as_float((254u - scode) << 23);   // 2^(127 - scode), exact
#pragma unroll
  for (int i = 0; i < kChunkValues; ++i) x[i] *= inv;
  // The signs: bytes 1 and 3 of the words of two values each, or the top bytes of the floats.
  uint32_t signs[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (SHIFT) {
      const uint32_t a = __builtin_amdgcn_perm(__float_as_uint(x[4 * i + 1]),
                                               __float_as_uint(x[4 * i]), 0x0c0c0703u);
      const uint32_t b = __builtin_amdgcn_perm(__float_as_uint(x[4 * i + 3]),
                                               __float_as_uint(x[4 * i + 2]), 0x0c0c0703u);
      signs[i] = b << 16 | a;
    } else {
      signs[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x07050301u);
    }
  }
  out = u32x2{e4m3_codes(x, signs[0]), e4m3_codes(x + 4, signs[1])};
}

// blockIdx.y (in steps of gridDim.y) is the group of rows that shares a shift vector (one
// group without SHIFT), blockIdx.x a run of kThreads * kChunks chunks of that group; thread
// t takes chunks t, t + kThreads, ... of the run.  chunks_per_row is a multiple of 4, so
// blocks never straddle groups and a quad of lanes is in range together.
//
// What bounds it: HBM, 3.03 bytes moved per value.  One thread per block with the codes
// formed by integer arithmetic (about 20 operations per value, strided 16-byte loads) was
// bound by the VALU instead: 720p K or Q
// (40 x 75600 x 128, 1.17 GB) 232 us, now 204 (5.8 TB/s); with a shift 277, now 204.
template <bool SHIFT>
__global__ __launch_bounds__(kThreads) void quantize_mxfp8_kernel(
    const u32x4* __restrict__ src, u32x2* __restrict__ codes, uint8_t* __restrict__ scales,
    long long n_chunks, const float* __restrict__ shift, uint32_t chunks_per_row,
    long long group_chunks) {
  const long long first = (long long)blockIdx.x * (kThreads * kChunks) + threadIdx.x;
  for (long long g = blockIdx.y; g * group_chunks < n_chunks; g += gridDim.y) {
    const long long base = g * group_chunks;
    const long long count = min(group_chunks, n_chunks - base);
    u32x4 w[kChunks];
#pragma unroll
    for (int u = 0; u < kChunks; ++u)
      w[u] = first + u * kThreads < count ? src[base + first + u * kThreads] : u32x4{0, 0, 0, 0};
    float sh[kChunkValues];
    uint32_t col = 0;
    if constexpr (SHIFT) col = (uint32_t)(first % chunks_per_row);
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
      if constexpr (SHIFT) {
        // The column advances by kThreads per chunk: rows of 32, 64, ... 2048 values come
        // back to the same one, so their shift is loaded once.
        if (u == 0 || kThreads % chunks_per_row != 0) {
          const float4* s4 = reinterpret_cast<const float4*>(
              shift + (g * chunks_per_row + col) * kChunkValues);
          const float4 a = s4[0], b = s4[1];
          sh[0] = a.x; sh[1] = a.y; sh[2] = a.z; sh[3] = a.w;
          sh[4] = b.x; sh[5] = b.y; sh[6] = b.z; sh[7] = b.w;
          col = (col + kThreads) % chunks_per_row;
        }
      }
      u32x2 out;
      uint32_t scode;
      quantize_chunk<SHIFT>(w[u], sh, out, scode);
      const long long chunk = first + u * kThreads;
      if (chunk < count) {
        codes[base + chunk] = out;
        if ((threadIdx.x & 3) == 0) scales[(base + chunk) >> 2] = (uint8_t)scode;
      }
    }
  }
}

// Several short groups a workgroup: blockIdx.x takes `groups` whole groups (groups *
// group_chunks <= kThreads * kChunks), and a thread finds each chunk's group and column by
// exact multiplications with rounded-up 2^32 / group_chunks and 2^32 / chunks_per_row (the
// divisors are at least 4, they and the dividends below 2^11).
//
// Why: with a workgroup a group, a shift per row of 128 values (16 chunks) left 1008 of 1024
// chunk places idle: 3024000 such rows 2418 us, now 468 (5.8 TB/s; 75600 rows 70.6, now 11.6;
// one thread a block took 486 and 15.1).  Source and codes pass by the caches that a shift
// vector's two halves are read through (without: 516).  At one group a workgroup (33 rows of
// 128, 215 us, 267 before) quantize_mxfp8_kernel does as well, so the line lies at two.
__global__ __launch_bounds__(kThreads) void quantize_mxfp8_short_kernel(
    const u32x4* __restrict__ src, u32x2* __restrict__ codes, uint8_t* __restrict__ scales,
    long long n_chunks, const float* __restrict__ shift, uint32_t chunks_per_row,
    uint32_t group_chunks, uint32_t groups, uint32_t row_magic, uint32_t group_magic) {
  const long long base_group = (long long)blockIdx.x * groups;
  const long long base = base_group * group_chunks;
  const uint32_t count =
      (uint32_t)min((long long)(groups * group_chunks), n_chunks - base);
  u32x4 w[kChunks];
#pragma unroll
  for (int u = 0; u < kChunks; ++u) {
    const uint32_t at = threadIdx.x + u * kThreads;
    w[u] = at < count ? __builtin_nontemporal_load(&src[base + at]) : u32x4{0, 0, 0, 0};
  }
  const float4* vectors = reinterpret_cast<const float4*>(shift) + 2 * base_group * chunks_per_row;
  float4 s4[kChunks][2];
#pragma unroll
  for (int u = 0; u < kChunks; ++u) {
    const uint32_t at = threadIdx.x + u * kThreads < count ? threadIdx.x + u * kThreads : 0;
    const uint32_t group = __umulhi(at, group_magic);
    const uint32_t rest = at - group * group_chunks;
    const uint32_t col = rest - __umulhi(rest, row_magic) * chunks_per_row;
    const uint32_t vec = 2 * (group * chunks_per_row + col);
    s4[u][0] = vectors[vec];
    s4[u][1] = vectors[vec + 1];
  }
#pragma unroll
  for (int u = 0; u < kChunks; ++u) {
    const uint32_t at = threadIdx.x + u * kThreads;
    const float4 a = s4[u][0], b = s4[u][1];
    const float sh[kChunkValues] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    u32x2 out;
    uint32_t scode;
    quantize_chunk<true>(w[u], sh, out, scode);
    if (at < count) {
      __builtin_nontemporal_store(out, &codes[base + at]);
      if ((threadIdx.x & 3) == 0) scales[(base + at) >> 2] = (uint8_t)scode;
    }
  }
}

// Mean over the N keys of every head.  A workgroup takes one column group of a head:
// kMeanCols columns (64 bytes of every row; all of a row when d is smaller).  Thread t
// sums 16-byte chunk t % C of rows t / C, t / C + P, ... (C chunks per group, P =
// kMeanThreads / C rows in flight per step, kMeanUnroll steps' loads issued together); then
// the P partial sums of every column are added in row order from LDS.  The order is fixed,
// so repeated calls agree bit for bit.
//
// What bounds it: HBM at many heads, and at few heads the loads one workgroup can keep in
// flight.  A head's column groups share 128-byte lines, so they go to the same XCD (L2), one
// after the other in its dispatch order (720p K, 774 MB: 222 us, now 196).
constexpr int kMeanThreads = 256;
constexpr int kMeanCols = 32;
constexpr int kMeanUnroll = 8;
constexpr int kMeanPhases = kMeanThreads / (kMeanCols / 8);   // partial sums for d >= 32
constexpr int kXcds = 8;       // accelerator dies; workgroups are dealt to them round-robin
// Fewer heads than this leave most XCDs idle in that order; their column groups go to one XCD
// each instead.  Measured as an XCD a head -> spread, us: 1 x 32760 x 128 39 -> 28, 1 x 16384 x
// 256 22.5 -> 14.3, 3 x 8192 x 256 9.1 -> 8.3; 5 x 16384 x 128 the other way, 15.4 -> 21.6.
constexpr int kMeanSpreadHeads = 4;

__global__ __launch_bounds__(kMeanThreads) void key_mean_kernel(const u32x4* __restrict__ k,
                                                                float* __restrict__ mean,
                                                                int bh, int N, int d,
                                                                bool spread) {
  __shared__ float part[kMeanThreads * 8];
  const int cols = d < kMeanCols ? d : kMeanCols;
  const int log_groups = __builtin_ctz(d) - __builtin_ctz(cols);   // powers of two
  const int slot = (int)(spread ? blockIdx.x : blockIdx.x / kXcds);   // place in the order
  const int group = slot & ((1 << log_groups) - 1);
  int head = slot >> log_groups;
  if (!spread) head = head * kXcds + (int)(blockIdx.x % kXcds);
  if (head >= bh) return;
  const int cpg = cols >> 3;                 // 16-byte chunks per group and row
  const int cpr = d >> 3;                    // chunks per row
  const int par = kMeanThreads / cpg;        // rows per step
  const int t = threadIdx.x;
  const int c = t % cpg;
  const u32x4* base = k + (size_t)head * (size_t)N * cpr + (size_t)group * cpg + c;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  auto add = [&](const u32x4& x) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[2 * j] += bf16_lo(x[j]);
      acc[2 * j + 1] += bf16_hi(x[j]);
    }
  };
  int r = t / cpg;
  for (; r + (kMeanUnroll - 1) * par < N; r += kMeanUnroll * par) {
    u32x4 x[kMeanUnroll];
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u) x[u] = base[(size_t)(r + u * par) * cpr];
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u) add(x[u]);
  }
  if (r < N) {   // the rest in one batch too; adding -0 changes no sum
    u32x4 x[kMeanUnroll];
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u)
      x[u] = u * par < N - r ? base[(size_t)(r + u * par) * cpr]
                             : u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u) add(x[u]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) part[t * 8 + i] = acc[i];
  __syncthreads();
  const float inv_n = 1.0f / (float)N;
  for (int e = t; e < cols; e += kMeanThreads) {
    const int ch = e >> 3, i = e & 7;
    float sum = 0.f;
    for (int rl = 0; rl < par; rl += 32) {   // par is 64 to 256: 32 reads in flight
      float x[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) x[u] = part[((rl + u) * cpg + ch) * 8 + i];
#pragma unroll
      for (int u = 0; u < 32; ++u) sum += x[u];
    }
    mean[(size_t)head * d + (size_t)group * cols + e] = sum * inv_n;
  }
}

// The same sums with a head's rows spread over d / 4 workgroups of one wave, for which the
// caller provides memory.  A lane takes four columns (8 bytes) of the rows of one phase p
// (p, p + kMeanPhases, ...), a wave 256 / d phases over all columns, so that it reads whole
// rows; the sums of a phase and their final order are those of key_mean_kernel, and so are
// the bits.
//
// Why: a workgroup of key_mean_kernel reads at about 25 GB/s however many loads it has in
// flight (line fills of its CU: each 64-byte piece brings in a whole line), and a head has
// only four.  40 heads of 75600 keys: 196 us against 126 (6.1 TB/s); 5 heads of 32760: 40
// against 24.  The second launch is paid back from about 8192 keys on with few heads (1 to 8:
// 8.2 against 7.3 us) and later with many (40 x 12000: 20.6 against 23.2; 40 x 16384: 26.7 both;
// 64 x 16384 39.4 against 41.6, the worst above the line).  kMeanSplitRows is where most head
// counts gain by a quarter or more.
constexpr int kMeanSplitUnroll = 16;
constexpr int kMeanSplitRows = 16384;

__global__ __launch_bounds__(64) void key_mean_phases_kernel(const u32x2* __restrict__ k,
                                                             float4* __restrict__ part, int N,
                                                             int d) {
  const int lpr = d >> 2;                    // lanes per row; also workgroups per head
  const int t = threadIdx.x;
  const int c = t % lpr;
  const int phase = (int)blockIdx.x * (64 / lpr) + t / lpr;
  const size_t head = blockIdx.y;
  const u32x2* base = k + head * (size_t)N * lpr + c;
  float4 acc{0.f, 0.f, 0.f, 0.f};
  auto add = [&](const u32x2& x) {
    acc.x += bf16_lo(x[0]);
    acc.y += bf16_hi(x[0]);
    acc.z += bf16_lo(x[1]);
    acc.w += bf16_hi(x[1]);
  };
  int r = phase;
  for (; r + (kMeanSplitUnroll - 1) * kMeanPhases < N; r += kMeanSplitUnroll * kMeanPhases) {
    u32x2 x[kMeanSplitUnroll];
#pragma unroll
    for (int u = 0; u < kMeanSplitUnroll; ++u) x[u] = base[(size_t)(r + u * kMeanPhases) * lpr];
#pragma unroll
    for (int u = 0; u < kMeanSplitUnroll; ++u) add(x[u]);
  }
  for (; r < N; r += kMeanPhases) add(base[(size_t)r * lpr]);
  part[(head * kMeanPhases + phase) * (size_t)lpr + c] = acc;
}

// mean[head][col] from the phase sums [head][kMeanPhases][d], added in phase order.
__global__ __launch_bounds__(64) void key_mean_join_kernel(const float* __restrict__ part,
                                                           float* __restrict__ mean, int N, int d,
                                                           int n_cols) {
  const int e = (int)(blockIdx.x * 64 + threadIdx.x);     // column of all heads' columns
  if (e >= n_cols) return;
  const size_t head = (size_t)(e / d);
  const float* p = part + head * kMeanPhases * d + (e - head * d);
  float x[kMeanPhases];
#pragma unroll
  for (int u = 0; u < kMeanPhases; ++u) x[u] = p[(size_t)u * d];
  const float inv_n = 1.0f / (float)N;
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < kMeanPhases; ++u) sum += x[u];
  mean[e] = sum * inv_n;
}

}  // namespace

hipError_t launch_quantize_mxfp8(const void* src, void* codes, void* scales,
                                 long long n_blocks, const float* shift, int blocks_per_row,
                                 long long group_rows, hipStream_t stream) {
  const long long n_chunks = n_blocks * 4;
  const long long cpr = (long long)blocks_per_row * 4;
  // Without a shift the whole array is one group; a group longer than the array is too.
  const long long rows = n_blocks / blocks_per_row;
  const bool one = shift == nullptr || group_rows >= rows;
  const long long group_chunks = one ? n_chunks : group_rows * cpr;
  const long long groups = (n_chunks + group_chunks - 1) / group_chunks;
  if (!one && 2 * group_chunks <= kThreads * kChunks) {   // at least two groups a workgroup
    const long long per = kThreads * kChunks / group_chunks;
    const auto magic = [](long long x) { return (uint32_t)(((1ull << 32) + x - 1) / x); };
    hipLaunchKernelGGL(quantize_mxfp8_short_kernel, dim3((unsigned)((groups + per - 1) / per)),
                       dim3(kThreads), 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x2*>(codes), static_cast<uint8_t*>(scales), n_chunks, shift,
                       (uint32_t)cpr, (uint32_t)group_chunks, (uint32_t)per, magic(cpr),
                       magic(group_chunks));
    return hipGetLastError();
  }
  const long long runs = (group_chunks + kThreads * kChunks - 1) / (kThreads * kChunks);
  const dim3 grid((unsigned)runs, (unsigned)(groups < 65535 ? groups : 65535));
  if (shift == nullptr)
    hipLaunchKernelGGL(quantize_mxfp8_kernel<false>, grid, dim3(kThreads), 0, stream,
                       static_cast<const u32x4*>(src), static_cast<u32x2*>(codes),
                       static_cast<uint8_t*>(scales), n_chunks, shift, (uint32_t)cpr,
                       group_chunks);
  else
    hipLaunchKernelGGL(quantize_mxfp8_kernel<true>, grid, dim3(kThreads), 0, stream,
                       static_cast<const u32x4*>(src), static_cast<u32x2*>(codes),
                       static_cast<uint8_t*>(scales), n_chunks, shift, (uint32_t)cpr,
                       group_chunks);
  return hipGetLastError();
}

size_t key_mean_split_bytes(int bh, int N, int d) {
  if (bh <= 0 || N < kMeanSplitRows || d < kMeanCols || d > 256) return 0;
  return (size_t)bh * kMeanPhases * (size_t)d * sizeof(float);
}

hipError_t launch_key_mean(const void* k, float* mean, int bh, int N, int d, float* split,
                           hipStream_t stream) {
  if (split != nullptr) {
    const int n_cols = bh * d;
    hipLaunchKernelGGL(key_mean_phases_kernel, dim3((unsigned)(d / 4), (unsigned)bh), dim3(64), 0,
                       stream, static_cast<const u32x2*>(k), reinterpret_cast<float4*>(split), N,
                       d);
    hipLaunchKernelGGL(key_mean_join_kernel, dim3((unsigned)((n_cols + 63) / 64)), dim3(64), 0,
                       stream, split, mean, N, d, n_cols);
    return hipGetLastError();
  }
  const int groups = d < kMeanCols ? 1 : d / kMeanCols;
  const bool spread = bh < kMeanSpreadHeads;
  const long long grid = (long long)(spread ? bh : (bh + kXcds - 1) / kXcds * kXcds) * groups;
  hipLaunchKernelGGL(key_mean_kernel, dim3((unsigned)grid), dim3(kMeanThreads), 0, stream,
                     static_cast<const u32x4*>(k), mean, bh, N, d, spread);
  return hipGetLastError();
}

}  // namespace dsattn

// The activation quantiser as a function that allocates nothing: device rows in, E4M3 codes and
// one scale per row out, any row length.  Rows of up to ROW_MAX elements are held in the registers
// of the threads that own them, in one launch.  A longer row is split over workgroups; the per-row absolute
// maxima they combine live in a file-scope device array, so the call needs no model, no
// workspace and no allocation of any kind (callers under HIP graph capture, serving loops and
// harnesses that may not allocate).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <mutex>
#include "../../include/pahq.h"
#include "device_util.h"

namespace pahq {

// One word per row: the bit pattern of max |x| over the row (non-negative floats order like
// unsigned integers, so atomicMax on the bits is exact and independent of the order of arrival).
// Every GPU the library runs on holds its own copy of this array until the process ends.
static __device__ __align__(256) unsigned scratch[PAHQ_NOALLOC_MAX_ROWS];

constexpr int CHUNK = 4096;          // elements of a row per workgroup (256 threads x 16)

__global__ __launch_bounds__(256) void noalloc_clear_k(unsigned* amax, int rows) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i < rows) amax[i] = 0u;
}

__global__ __launch_bounds__(256) void noalloc_amax_k(const float* x, int cols, unsigned* amax) {
  const int row = blockIdx.y;
  const float* p = x + (long long)row * cols;
  const int e0 = blockIdx.x * CHUNK, e1 = min(cols, e0 + CHUNK);
  float m = 0.f;
  for (int e = e0 + threadIdx.x; e < e1; e += 256) m = fmaxf(m, fabsf(p[e]));
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) atomicMax(&amax[row], __float_as_uint(m));
}

__global__ __launch_bounds__(256) void noalloc_encode_k(const float* x, int cols, const unsigned* amax,
                                                        uint8_t* codes, float* scales) {
  const int row = blockIdx.y;
  const float am = __uint_as_float(amax[row]);
  const float scale = (am == 0.f) ? 1.0f : am / 448.0f;
  const float inv = 1.0f / scale;
  const float* p = x + (long long)row * cols;
  uint8_t* o = codes + (long long)row * cols;
  const int e0 = blockIdx.x * CHUNK, e1 = min(cols, e0 + CHUNK);
  for (int e = e0 + threadIdx.x; e < e1; e += 256) o[e] = (uint8_t)e4m3_encode(p[e] * inv);
  if (blockIdx.x == 0 && threadIdx.x == 0) scales[row] = scale;
}

// One row in the registers of NT threads, read once and encoded from there (HBM-bound: five bytes per element).
// A thread takes up to four groups of four neighbouring elements.  Groups start where the row's codes reach a word
// boundary, so that four codes leave as one word whatever the row length is; the up to three elements in front of the
// first group and behind the last go one to a thread.  The 16-byte loads need the alignment of a float only.
// NT = 64 puts four rows into a workgroup of four waves, which never meet.  3001 rows of 3072: 23.6 -> 8.3 us (5.5 TB/s)
// against the clear, maximum and encode launches below, which read the row twice and store single bytes.
struct __attribute__((packed, aligned(4))) f4u { float x, y, z, w; };
template <int NT>
__global__ __launch_bounds__(NT < 256 ? 256 : NT) void noalloc_row_k(const float* x, int rows, int cols, uint8_t* codes, float* scales) {
  constexpr int Q = 4;
  const int row = NT == 64 ? (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6) : (int)blockIdx.x;
  const int t = NT == 64 ? threadIdx.x & 63 : threadIdx.x;
  if (NT == 64 && row >= rows) return;               // (a wave owns its row: no barrier follows)
  const float* p = x + (long long)row * cols;
  uint8_t* o = codes + (long long)row * cols;
  const int head = min((int)(-(uintptr_t)o & 3), cols), nq = (cols - head) >> 2, tail = head + 4 * nq;
  float v[Q][4];
  float m = 0.f;
#pragma unroll
  for (int q = 0; q < Q; q++) {
    const int g = q * NT + t;
    v[q][0] = v[q][1] = v[q][2] = v[q][3] = 0.f;
    if (g < nq) { const f4u w = *(const f4u*)(p + head + 4 * g); v[q][0] = w.x; v[q][1] = w.y; v[q][2] = w.z; v[q][3] = w.w; }
  }
  // this thread's single element, if it has one
  const int e1 = t < head ? t : (t >= 4 && tail + t - 4 < cols ? tail + t - 4 : -1);
  const float v1 = e1 >= 0 ? p[e1] : 0.f;
#pragma unroll
  for (int q = 0; q < Q; q++)
#pragma unroll
    for (int c = 0; c < 4; c++) m = fmaxf(m, fabsf(v[q][c]));
  m = wave_max(fmaxf(m, fabsf(v1)));
  if (NT > 64) {
    __shared__ float part[NT / 64];
    if ((t & 63) == 0) part[t >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; w++) m = fmaxf(m, part[w]);
  }
  const float scale = (m == 0.f) ? 1.0f : m / 448.0f;
  const float inv = 1.0f / scale;
#pragma unroll
  for (int q = 0; q < Q; q++) {
    const int g = q * NT + t;
    if (g < nq) *(uint32_t*)(o + head + 4 * g) = e4m3_encode4(v[q][0] * inv, v[q][1] * inv, v[q][2] * inv, v[q][3] * inv);
  }
  if (e1 >= 0) o[e1] = (uint8_t)e4m3_encode(v1 * inv);
  if (t == 0) scales[row] = scale;
}
constexpr int ROW_MAX = 1024 * 16;                   // elements of a row 1024 threads hold

namespace {
constexpr int MAX_DEVICES = 64;
unsigned* scratch_ptr[MAX_DEVICES];      // device address of `scratch` on each GPU (its name is a host-side stand-in)
std::mutex scratch_mu;

// Address of this device's copy of the array, looked up once per device with that device current.
int scratch_of_current_device(unsigned** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return PAHQ_EHIP;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PAHQ_EHIP;
    scratch_ptr[dev] = (unsigned*)p;
  }
  *out = scratch_ptr[dev];
  return PAHQ_OK;
}
}  // namespace

}  // namespace pahq

extern "C" int pahq_quantize_rows_noalloc(void* hip_stream, const float* x, int32_t rows, int32_t cols,
                                          uint8_t* codes, float* scales) {
  using namespace pahq;
  if (rows < 0 || cols < 1) return PAHQ_EINVAL;
  if (rows > PAHQ_NOALLOC_MAX_ROWS) return PAHQ_ETOOBIG;
  if (rows == 0) return PAHQ_OK;
  if (!x || !codes || !scales) return PAHQ_EINVAL;
  if (cols <= ROW_MAX) {
    // the fewest threads whose registers hold the row: 16 elements each
    hipStream_t st = (hipStream_t)hip_stream;
    if (cols <= 64 * 16) hipLaunchKernelGGL(noalloc_row_k<64>, dim3((rows + 3) / 4), dim3(256), 0, st, x, rows, cols, codes, scales);
    else if (cols <= 256 * 16) hipLaunchKernelGGL(noalloc_row_k<256>, dim3(rows), dim3(256), 0, st, x, rows, cols, codes, scales);
    else hipLaunchKernelGGL(noalloc_row_k<1024>, dim3(rows), dim3(1024), 0, st, x, rows, cols, codes, scales);
    return hipGetLastError() == hipSuccess ? PAHQ_OK : PAHQ_EHIP;
  }
  unsigned* amax = nullptr;
  int rc = scratch_of_current_device(&amax);
  if (rc != PAHQ_OK) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  // the array keeps the last call's maxima: the rows of this call start from zero (a fill kernel,
  // not a memset, so that the sequence can be captured into a graph)
  hipLaunchKernelGGL(noalloc_clear_k, dim3((rows + 255) / 256), dim3(256), 0, st, amax, rows);
  const dim3 grid((cols + CHUNK - 1) / CHUNK, rows);
  hipLaunchKernelGGL(noalloc_amax_k, grid, dim3(256), 0, st, x, cols, amax);
  hipLaunchKernelGGL(noalloc_encode_k, grid, dim3(256), 0, st, x, cols, amax, codes, scales);
  return hipGetLastError() == hipSuccess ? PAHQ_OK : PAHQ_EHIP;
}

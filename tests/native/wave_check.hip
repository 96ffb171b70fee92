// Device check of the wave-wide routines (test helper, built by build()): each
// case is run by one wave or one workgroup on data the test supplies.
#include <hip/hip_runtime.h>

#include "../../paper_2404_10404_amd/csrc/fr_row.hpp"
#include "../../paper_2404_10404_amd/csrc/sha256_wave.hpp"

using namespace gkr;

namespace {

// One workgroup of two waves per case: the chaining value after `rounds`
// compressions of the case's blocks, from the value in st. With helped, wave 1
// writes the schedules.
__global__ void __launch_bounds__(128) k_sha_chain(const uint32_t* st, const uint32_t* blocks, uint32_t* out,
                                                   uint32_t rounds, int helped) {
  __shared__ __attribute__((aligned(16))) ShaBuf buf;
  __shared__ ShaHelper help;
  const uint32_t wid = threadIdx.x >> 6;
  const uint32_t* blk = blocks + 16ull * rounds * blockIdx.x;
  ShaLanes s;
  if (wid == 0) {
    s = sha_lanes_load(st + 8ull * blockIdx.x);
    sha_init(&buf);
    if (threadIdx.x == 0) help.ready = 0;
  }
  __syncthreads();
  for (uint32_t r = 0; r < rounds; ++r) {
    const uint32_t w = blk[16 * r + (threadIdx.x & 15)];
    if (wid == 0) s = helped ? sha_compress_wave<true>(s, w, &buf, &help, 3 * r) : sha_compress_wave<false>(s, w, &buf);
    else if (helped) sha_help(w, &buf, &help, 3 * r);
    __syncthreads();
  }
  if (wid == 0) sha_lanes_store(out + 8ull * blockIdx.x, s);
}

// One wave per case: SHA-256 of `len` words (9, 11 or 17).
__global__ void __launch_bounds__(64) k_sha_message(const uint32_t* msg, uint32_t* out, int len) {
  __shared__ __attribute__((aligned(16))) ShaBuf buf;
  sha_init(&buf);
  if (threadIdx.x < (uint32_t)len) buf.msg[threadIdx.x] = msg[(uint64_t)len * blockIdx.x + threadIdx.x];
  const ShaLanes s = len == 9 ? sha_message_wave<9>(&buf) : len == 11 ? sha_message_wave<11>(&buf) : sha_message_wave<17>(&buf);
  sha_lanes_store(out + 8ull * blockIdx.x, s);
}

// Four cases per wave, a row of 16 lanes each: the quadratic (v0, v1, c2) at r, from
// 32 words per case (r, v0, v1, c2).
__global__ void __launch_bounds__(64) k_row_quadratic(const uint32_t* in, uint32_t* out) {
  const uint32_t i = threadIdx.x & 15;
  const uint64_t k = 4ull * blockIdx.x + (threadIdx.x >> 4);
  const uint32_t* c = in + 32 * k;
  uint32_t r[8];
  for (int j = 0; j < 8; ++j) r[j] = c[j];
  const uint32_t e = row_quadratic(r, i < 8 ? c[8 + i] : 0, i < 8 ? c[16 + i] : 0, i < 8 ? c[24 + i] : 0);
  if (i < 8) out[8 * k + i] = e;
}

}  // namespace

extern "C" int wavecheck_row_quadratic(const void* d_in, void* d_out, uint32_t waves) {
  if (!d_in || !d_out || waves < 1 || waves > 4096) return -1;
  k_row_quadratic<<<waves, 64>>>(static_cast<const uint32_t*>(d_in), static_cast<uint32_t*>(d_out));
  return hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess ? -3 : 0;
}

// Synchronous; 0, -1 for bad arguments, -3 when the launch fails.
extern "C" int wavecheck_sha_chain(const void* d_st, const void* d_blocks, void* d_out, uint32_t cases, uint32_t rounds,
                                   int helped) {
  if (!d_st || !d_blocks || !d_out || cases < 1 || cases > 4096 || rounds < 1 || rounds > 64) return -1;
  k_sha_chain<<<cases, 128>>>(static_cast<const uint32_t*>(d_st), static_cast<const uint32_t*>(d_blocks),
                              static_cast<uint32_t*>(d_out), rounds, helped);
  return hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess ? -3 : 0;
}

extern "C" int wavecheck_sha_message(const void* d_msg, void* d_out, uint32_t cases, int len) {
  if (!d_msg || !d_out || cases < 1 || cases > 4096 || (len != 9 && len != 11 && len != 17)) return -1;
  k_sha_message<<<cases, 64>>>(static_cast<const uint32_t*>(d_msg), static_cast<uint32_t*>(d_out), len);
  return hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess ? -3 : 0;
}

// The phase-2 copy contraction on the matrix cores (Section 2.3, phase 2 of a
// data-parallel layer with the copy factors kept apart): for every
// sub-circuit wire y,
//   P[y] = sum_c U[c] W[y,c] R^-1 mod p,   Q[y] = sum_c V[c] W[y,c] R^-1 mod p
// (Montgomery forms), the same values the scalar contraction computes with
// lazy Montgomery products.
//
// The sums are exact integer sums of byte products. With W_j, U_i the bytes
// of W[y,c] and U[c] (little endian, 32 each),
//   sum_c U[c] W[y,c] = sum_k 2^(8k) E_k,  E_k = sum_c sum_{i + j = k} U_i[c] W_j[y,c],
// which is one matrix product: A[y][(c,j)] = W_j[y,c] is the table itself
// (row y is 32 * 2^n consecutive bytes), and B[(c,j)][k] = U_(k-j)[c] (zero
// outside 0 <= k - j < 32) is a banded matrix built from U. Columns 0..62 of
// B hold the bands of U, 64..126 those of V, 63 is all ones (the row sums).
// The int8 matrix instructions multiply signed bytes: both operands are
// offset by 128 (a byte u is stored as u - 128), and
//   sum a_u b_u = sum a_s b_s + 128 sum_K a_s + 128 sum_K b_u,
// where sum_K a_s is the all-ones column and sum_K b_u follows from the byte
// sums of U and V. Each workgroup takes 128 rows and one chunk of K
// (at most 2^15 bytes: |sum a_s b_s| < 2^29 fits the 32-bit accumulators) and
// stores its partial columns; the epilogue adds the chunks, applies the
// offsets, assembles the integer per row and reduces it (cc_sum.hpp).
#include <string.h>

#include <algorithm>

#include "cc_sum.hpp"
#include "gkr_bodies.hpp"
#include "gkr_contract.hpp"
#include "gkr_profile.hpp"
#include "gkr_program.hpp"

namespace gkr {

typedef int I32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kCcCols = 128;        // B columns: two vectors of 63 bands, the ones column, one unused
constexpr uint32_t kCcOnes = 63;         // the all-ones column
constexpr uint32_t kCcRows = 256;        // rows per workgroup (eight waves of two 16-row groups)
constexpr uint32_t kCcThreads = 512;
constexpr uint32_t kCcBlockK = 256;      // K bytes staged in LDS at a time (four 64-byte steps)
constexpr uint32_t kCcLdsStride = 272;   // bytes per staged column: 16 lanes of one read hit distinct banks
constexpr uint32_t kCcMaxChunkK = 1u << 15;

// ST_CC_BUILD: the banded matrix, stored transposed (Bt[col][K], int8 with
// the 128 offset). Thread t: column t >> n, copy c = t & (2^n - 1), 32 bytes.
// p0 U, p1 V, p2 Bt; u0 n; q0 2^n * 128.
__global__ void __launch_bounds__(kBlock) k_cc_build(Step st) {
  const Fr* U = P<const Fr*>(st, 0);
  const Fr* V = P<const Fr*>(st, 1);
  uint8_t* Bt = P<uint8_t*>(st, 2);
  const uint32_t n = st.u[0];
  const uint64_t K = 32ull << n;
  for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < st.q[0];
       t += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t col = (uint32_t)(t >> n);
    const uint64_t c = t & ((1ull << n) - 1);
    uint32_t out[8];
    if (col == kCcOnes) {
#pragma unroll
      for (int d = 0; d < 8; ++d) out[d] = 0x01010101u;
    } else if (col == kCcCols - 1) {
#pragma unroll
      for (int d = 0; d < 8; ++d) out[d] = 0;
    } else {
      const Fr x = ldf(col < kCcOnes ? U : V, c);
      const int k = (int)(col < kCcOnes ? col : col - 64);
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = k - (4 * d + e);  // byte i of x meets byte j = 4d + e of W
          uint32_t b = 0;
          if (i >= 0 && i < 32) b = (x.v[i >> 2] >> (8 * (i & 3))) & 0xffu;
          word |= ((b - 128u) & 0xffu) << (8 * e);
        }
        out[d] = word;
      }
    }
    GlobalU4* q = (GlobalU4*)(Bt + (uint64_t)col * K + 32 * c);
    q[0] = U32x4{out[0], out[1], out[2], out[3]};
    q[1] = U32x4{out[4], out[5], out[6], out[7]};
  }
}

// ST_CC_BSUM: byte sums BS[v * 32 + i] = sum_c byte i of (v ? V : U)[c]; one
// workgroup per (v, i). p0 U, p1 V, p2 BS; q0 2^n.
__global__ void __launch_bounds__(kBlock) k_cc_bsum(Step st) {
  const uint32_t v = blockIdx.x >> 5, i = blockIdx.x & 31;
  const uint32_t* X = P<const uint32_t*>(st, v);
  uint32_t s = 0;
  for (uint64_t c = threadIdx.x; c < st.q[0]; c += kBlock) s += (X[8 * c + (i >> 2)] >> (8 * (i & 3))) & 0xffu;
  __shared__ uint32_t red[kBlock / 64];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += (uint32_t)__shfl_xor((int)s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kBlock / 64; ++w) t += red[w];
    P<uint32_t*>(st, 2)[blockIdx.x] = t;
  }
}

// ST_CC_GEMM: partial column sums of 256 rows over one K chunk. Workgroup b:
// chunk b / row_tiles, rows 256 (b mod row_tiles) ..; wave w takes the
// 16-row groups 2w and 2w + 1 against all eight 16-column groups. Lane l
// holds 16 bytes of row (l mod 16) and of column (l mod 16) at K offset
// 16 (l / 16) of each 64-byte step (the instruction sums the four lane groups),
// and receives rows 4 (l / 16) .. + 3 of column l mod 16.
// Term i of row y is 32 bytes at y q2 + i q3 of W: q3 = 32 for sums along a
// table's rows (16 bytes per lane at a stride of one row; a row's lines are used
// whole over the block's four steps), q2 = 32 for sums down its columns (16
// rows' terms are 512 consecutive bytes).
// p0 W (bytes), p1 Bt, p2 part (int32 [chunk][row][128]); u0 n, u1 row_tiles;
// q0 chunk bytes, q1 rows, q2 row stride, q3 term stride (bytes).
__global__ void __launch_bounds__(kCcThreads) k_cc_gemm(Step st) {
  __shared__ __attribute__((aligned(16))) uint8_t Bs[kCcCols * kCcLdsStride];
  const uint8_t* W = P<const uint8_t*>(st, 0);
  const uint8_t* Bt = P<const uint8_t*>(st, 1);
  int32_t* part = P<int32_t*>(st, 2);
  const uint32_t n = st.u[0], row_tiles = st.u[1];
  const uint64_t K = 32ull << n, Kc = st.q[0], rows = st.q[1];
  const uint32_t chunk = blockIdx.x / row_tiles, rt = blockIdx.x - chunk * row_tiles;
  const uint64_t y0 = (uint64_t)rt * kCcRows, k0 = (uint64_t)chunk * Kc;
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const uint32_t nblk = (uint32_t)(Kc / kCcBlockK);
  // this thread's share of a staged block: column t / 4, 64 bytes at (t & 3) * 64
  const uint32_t scol = threadIdx.x >> 2, soff = (threadIdx.x & 3) * 64;
  const U32x4* bsrc = (const U32x4*)(Bt + (uint64_t)scol * K + k0 + soff);
  const U32x4* arow[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    arow[h] = (const U32x4*)(W + (y0 + (2 * wid + h) * 16 + r) * st.q[2] + (k0 / 32 + (g >> 1)) * st.q[3] + 16 * (g & 1));
  const uint64_t astep = 2 * st.q[3] / 16;  // vectors from one 64-byte step (two terms) to the next
  I32x4 acc[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int cg = 0; cg < 8; ++cg) acc[h][cg] = I32x4{0, 0, 0, 0};
  U32x4 bst[4], anext[2][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) bst[e] = bsrc[e];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int s = 0; s < 4; ++s) anext[h][s] = arow[h][s * astep];
  for (uint32_t blk = 0; blk < nblk; ++blk) {
    __syncthreads();  // every wave has finished the previous block's LDS reads
#pragma unroll
    for (int e = 0; e < 4; ++e) *(U32x4*)(Bs + scol * kCcLdsStride + soff + 16 * e) = bst[e];
    U32x4 a[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < 4; ++s) a[h][s] = anext[h][s];
    __syncthreads();
    if (blk + 1 < nblk) {
      const uint64_t adv = (uint64_t)(blk + 1) * (kCcBlockK / 16), aadv = 4 * (uint64_t)(blk + 1) * astep;
#pragma unroll
      for (int e = 0; e < 4; ++e) bst[e] = bsrc[adv + e];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 4; ++s) anext[h][s] = arow[h][aadv + s * astep];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int cg = 0; cg < 8; ++cg) {
        const U32x4 bv = *(const U32x4*)(Bs + (cg * 16 + r) * kCcLdsStride + 64 * s + 16 * g);
        const I32x4 bf = I32x4{(int)bv.x, (int)bv.y, (int)bv.z, (int)bv.w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          // W's bytes u as signed u - 128: the top bit of every byte flipped
          const I32x4 af = I32x4{(int)(a[h][s].x ^ 0x80808080u), (int)(a[h][s].y ^ 0x80808080u),
                                 (int)(a[h][s].z ^ 0x80808080u), (int)(a[h][s].w ^ 0x80808080u)};
          acc[h][cg] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af, bf, acc[h][cg], 0, 0, 0);
        }
      }
    }
  }
  // rows 4g .. 4g + 3 of each 16-row group, column cg * 16 + r
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int cg = 0; cg < 8; ++cg)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t y = y0 + (2 * wid + h) * 16 + 4 * g + e;
        part[((uint64_t)chunk * rows + y) * kCcCols + cg * 16 + r] = acc[h][cg][e];
      }
}

// ST_CC_EPILOGUE: a workgroup takes u1 rows, two for tables of few rows (which
// have many chunks: 2^9 rows, 128 chunks took 142 us with eight) and eight
// otherwise. All threads first add the chunks' partial columns, two rows of 128
// consecutive columns at a time, into shared memory; then one thread per (row,
// vector) takes the 63 band columns of its vector and the ones column, the offsets,
// the integer sum_k 2^(8k) E_k and its Montgomery reduction (cc_sum.hpp; w[0..7]
// 2^508 mod p). 2^14 rows take 18 us (57 with the two threads of a row also adding
// the chunks, 63 loads per chunk at a stride of a row).
// p0 part, p1 BS, p2 P out, p3 Q out; u0 chunks, u1 rows per workgroup; q0 rows.
constexpr uint32_t kCcEpiRows = 8;

__global__ void __launch_bounds__(kBlock) k_cc_epilogue(Step st) {
  __shared__ int64_t sums[kCcEpiRows][kCcCols + 1];
  __shared__ uint64_t ps[2][33];  // prefix sums of the vectors' byte sums
  const int32_t* part = P<const int32_t*>(st, 0);
  const uint32_t* BS = P<const uint32_t*>(st, 1);
  const uint32_t chunks = st.u[0];
  const uint32_t per = st.u[1];
  const uint64_t rows = st.q[0], y0 = (uint64_t)blockIdx.x * per;
  if (threadIdx.x < 2) {
    uint64_t s = 0;
    for (int i = 0; i < 32; ++i) {
      ps[threadIdx.x][i] = s;
      s += BS[32 * threadIdx.x + i];
    }
    ps[threadIdx.x][32] = s;
  }
  const uint32_t col = threadIdx.x & (kCcCols - 1);
  for (uint32_t q = 0; q < per; q += 2) {
    const uint32_t row = q + threadIdx.x / kCcCols;
    int64_t d = 0;
    if (y0 + row < rows) {
      const int32_t* src = part + (y0 + row) * kCcCols + col;
#pragma unroll 8
      for (uint32_t ch = 0; ch < chunks; ++ch) d += src[(uint64_t)ch * rows * kCcCols];
    }
    sums[row][col] = d;
  }
  __syncthreads();
  const uint32_t row = threadIdx.x >> 1, v = threadIdx.x & 1;
  if (threadIdx.x >= 2 * per || y0 + row >= rows) return;
  const int64_t rs = sums[row][kCcOnes];
  CcSum sum = cc_sum_zero();
#pragma unroll
  for (int k = 0; k < kCcBands; ++k) {
    // sum_K b_u of band k covers bytes max(0, k - 31) .. min(k, 31)
    const uint64_t cs = ps[v][k < 31 ? k + 1 : 32] - ps[v][k > 31 ? k - 31 : 0];
    cc_sum_band(sum, k, (uint64_t)(sums[row][64 * v + k] + 128 * rs + 128 * (int64_t)cs));
  }
  const Fr out = cc_sum_reduce(sum, st.w);
  Fr *ou = P<Fr*>(st, 2), *ov = P<Fr*>(st, 3);
  stf(v ? ov : ou, y0 + row, out);
}

void launch_cc_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles), block(kBlock);
  switch (st.type) {
    case ST_CC_BUILD: k_cc_build<<<grid, block, 0, s>>>(st); break;
    case ST_CC_BSUM: k_cc_bsum<<<grid, block, 0, s>>>(st); break;
    case ST_CC_GEMM: k_cc_gemm<<<grid, dim3(kCcThreads), 0, s>>>(st); break;
    case ST_CC_EPILOGUE: k_cc_epilogue<<<grid, block, 0, s>>>(st); break;
    default: break;
  }
  if (tok >= 0) prof_end(tok, s, PC_COPY_CONTRACT, st.bytes, st.mulmods);
}

// ---------------------------------------------------------------- host

bool cc_applies(uint32_t n, uint32_t sigma) { return n >= kCcMinLogCopies && sigma >= kCcMinLogRows; }

CcPlan cc_plan(uint32_t n, uint32_t sigma) {
  CcPlan cp;
  const uint64_t K = 32ull << n, rows = 1ull << sigma, row_tiles = rows / kCcRows;
  uint64_t chunks = (kCcTargetGroups + row_tiles - 1) / row_tiles;
  chunks = std::max<uint64_t>(chunks, K / kCcMaxChunkK);
  chunks = std::min<uint64_t>(chunks, K / kCcBlockK);
  uint64_t p2 = 1;
  while (p2 < chunks) p2 *= 2;
  cp.chunks = (uint32_t)p2;
  cp.chunk_bytes = K / p2;
  cp.row_tiles = (uint32_t)row_tiles;
  cp.bt_bytes = (size_t)kCcCols * K;
  cp.part_bytes = (size_t)p2 * rows * kCcCols * sizeof(int32_t);
  cp.bs_bytes = 64 * sizeof(uint32_t);
  return cp;
}

size_t cc_scratch_bytes(uint32_t n, uint32_t sigma) {
  if (!cc_applies(n, sigma)) return 0;
  const CcPlan cp = cc_plan(n, sigma);
  return cp.bt_bytes + cp.part_bytes + 256;
}

void* cc_scratch(const Workspace& w, uint32_t n, uint32_t sigma) {
  if (!cc_applies(n, sigma)) return nullptr;
  if (n >= kCcOwnLogCopies) return w.cc;
  const size_t room = 2 * sizeof(Fr) * (size_t)(w.H - w.G);  // H follows G and is as large
  return cc_scratch_bytes(n, sigma) <= room ? w.G : nullptr;
}

void emit_contract_mfma(Program& pg, const Fr* W, const Fr* U, const Fr* V, Fr* out_u, Fr* out_v, uint32_t log_terms,
                        uint32_t log_rows, bool transposed, void* scratch) {
  const uint32_t n = log_terms;
  const CcPlan cp = cc_plan(log_terms, log_rows);
  uint8_t* base = static_cast<uint8_t*>(scratch);
  uint8_t* Bt = base;
  int32_t* part = reinterpret_cast<int32_t*>(base + cp.bt_bytes);
  uint32_t* BS = reinterpret_cast<uint32_t*>(base + cp.bt_bytes + cp.part_bytes);
  const uint64_t rows = 1ull << log_rows, ncop = 1ull << log_terms;
  auto mk = [](uint32_t type, uint32_t tiles) {
    Step st;
    memset(&st, 0, sizeof(st));
    st.type = type;
    st.ntiles = tiles < 1 ? 1 : tiles;
    return st;
  };
  {
    const uint64_t t = ncop * kCcCols;
    Step st = mk(ST_CC_BUILD, (uint32_t)std::min<uint64_t>((t + kBlock - 1) / kBlock, 65535u * 8));
    st.p[0] = U; st.p[1] = V; st.p[2] = Bt; st.u[0] = n; st.q[0] = t;
    st.bytes = 64.0 * ncop + (double)cp.bt_bytes;
    pg.steps.push_back(st);
  }
  {
    Step st = mk(ST_CC_BSUM, 64);
    st.p[0] = U; st.p[1] = V; st.p[2] = BS; st.q[0] = ncop;
    st.bytes = 64.0 * ncop;
    pg.steps.push_back(st);
  }
  {
    Step st = mk(ST_CC_GEMM, cp.row_tiles * cp.chunks);
    st.p[0] = W; st.p[1] = Bt; st.p[2] = part; st.u[0] = n; st.u[1] = cp.row_tiles;
    st.q[0] = cp.chunk_bytes; st.q[1] = rows;
    st.q[2] = transposed ? 32 : 32 * ncop; st.q[3] = transposed ? 32 * rows : 32;
    st.bytes = 32.0 * (double)(rows << n) + (double)cp.part_bytes;  // no field products: int8 matrix work
    pg.steps.push_back(st);
  }
  {
    const uint32_t per = rows >= 4096 ? kCcEpiRows : 2;
    Step st = mk(ST_CC_EPILOGUE, (uint32_t)((rows + per - 1) / per));
    st.u[1] = per;
    st.p[0] = part; st.p[1] = BS; st.p[2] = out_u; st.p[3] = out_v; st.u[0] = cp.chunks; st.q[0] = rows;
    memcpy(st.w, kCcPow508, sizeof(kCcPow508));
    st.bytes = (double)cp.part_bytes + 64.0 * rows;
    st.mulmods = (double)rows;  // one reduction per row and vector
    pg.steps.push_back(st);
  }
}

}  // namespace gkr

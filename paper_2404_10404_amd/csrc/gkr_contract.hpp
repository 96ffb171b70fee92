// The phase-2 copy contraction on the matrix cores (gkr_contract.hip): plan,
// step emission and launcher. Used by the plain path for layers with at least
// 2^kCcMinLogRows sub-circuit wires and 2^kCcMinLogCopies copies; the scalar
// contraction (ST_COPY_CONTRACT) takes every other layer and the batch kernel.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "gkr_internal.hpp"

namespace gkr {

constexpr uint32_t kCcMinLogCopies = 9;   // rows of at least 16 KiB
constexpr uint32_t kCcOwnLogCopies = 10;  // from here on the workspace holds scratch of its own
constexpr uint32_t kCcMinLogRows = 8;     // at least one 256-row tile
constexpr uint64_t kCcTargetGroups = 256; // workgroups of the product (row tiles x K chunks), one per CU

struct CcPlan {
  uint32_t chunks = 0, row_tiles = 0;
  uint64_t chunk_bytes = 0;
  size_t bt_bytes = 0, part_bytes = 0, bs_bytes = 0;
};

bool cc_applies(uint32_t n, uint32_t sigma);
CcPlan cc_plan(uint32_t n, uint32_t sigma);
// Scratch bytes of one contraction (banded matrix, partial columns, byte sums); 0 if it does not apply.
size_t cc_scratch_bytes(uint32_t n, uint32_t sigma);

// Where a contraction over 2^n copies may put that scratch outside phase 1's rounds
// (null: it does not apply, or nowhere): with 2^9 copies in the tables G and H, where
// they are large enough. They are free then, and scratch of its own (36 MB for 2^19
// entries) would grow a workspace that has to fit gkr_prove_circuit_noalloc's array;
// where they are too small (2^19 entries or fewer) the scalar pass is the faster one
// (ten layers of 2^19 entries 6.19 ms, on the matrix cores 6.89).
void* cc_scratch(const Workspace& w, uint32_t n, uint32_t sigma);

struct Program;
// out_u[r] = sum_i U[i] X(r, i) R^-1 and out_v with V, for r < 2^log_rows over i <
// 2^log_terms, where X(r, i) is entry r 2^log_terms + i of W, or entry
// i 2^log_rows + r with `transposed` (sums over a table's rows instead of its
// columns); scratch holds cc_scratch_bytes(log_terms, log_rows) bytes, 256-byte aligned.
void emit_contract_mfma(Program& pg, const Fr* W, const Fr* U, const Fr* V, Fr* out_u, Fr* out_v, uint32_t log_terms,
                        uint32_t log_rows, bool transposed, void* scratch);
void launch_cc_step(const Step& st, hipStream_t s);

}  // namespace gkr

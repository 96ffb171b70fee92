// Phase 1 with the addition gates contracted over the copies (gkr_split.hip):
// used by the plain path for wide layers of many copies.
#pragma once

#include <cmath>

#include "gkr_internal.hpp"
#include "gkr_program.hpp"

namespace gkr {

// Whether a layer with mul_gates MUL gates whose next layer has 2^sigma wires in 2^n
// copies takes this form.
bool split_applies(uint32_t n, uint32_t sigma, uint64_t mul_gates);

// Phase 1 of a layer (tables, rounds, vx): W = V_{i+1}, rx the challenges,
// proof the layer's messages. Leaves EL (eq at the local part of rx) in w.EL and
// the phase-2 wiring tables Ma, Mb, Aa, Ab in w.P, w.Q, w.Ka, w.Kb.
void emit_phase1_split(Program& pg, const Workspace& w, const LayerWiring& lw, const Fr* W, uint32_t n, uint32_t sigma,
                       uint64_t gates, uint64_t mul_gates, Fr* rx, uint32_t* proof, const Tuning& tun);

// The phase-2 tables Fa, Fb, Ka, Kb, Ks from those wiring tables.
void emit_p2_final(Program& pg, const Workspace& w, uint64_t rows);

void launch_split_step(const Step& st, hipStream_t s);

// Expected share of the MUL table's rows that are not zero after j folds, for mul_gates
// gates with random left inputs over rows (for the work records only).
inline double split_active_share(uint64_t mul_gates, uint64_t rows, uint32_t j) {
  return 1.0 - std::exp(-(double)(1ull << j) * (double)mul_gates / (double)rows);
}

}  // namespace gkr

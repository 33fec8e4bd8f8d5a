// Wait counts of the many-row GEMM's LDS ring, apart from the kernel so that they compile on the host.
#pragma once

namespace dvi {

// The vector-memory operations of a wave that are certainly younger than its copies of the stage that it
// is about to read; waiting until no more than these are in flight serves every stage.
// Order of issue: the copies (PX each) of stages 0 .. NS - 2, then WD chunks of weights (RT loads each);
// from there per stage s the plain loop waits for stage s, copies stage s + NS - 1 and reloads the
// weights of its CPS chunks.  The piped loop waits for stage 0, copies stage NS - 1, and then per stage s
// reloads the weights of all chunks but the last, waits for stage s + 1, copies stage s + NS and reloads
// the last chunk's.
// Stages of the first NS - 1 copies have the first weights and NS - 2 stages' copies behind them (first);
// later ones NS - 2 stages' copies and (NS - 1) CPS chunks of weights (loop), but one chunk fewer for
// stage NS - 1 of the piped loop, whose copies go out before any reload.
constexpr int ring_wait_count(int CPS, int NS, int WD, int RT, int PX, bool piped) {
    const int loop = ((NS - 1) * CPS - (piped ? 1 : 0)) * RT + (NS - 2) * PX;
    const int first = WD * RT + (NS - 2) * PX;
    const int n = loop < first ? loop : first;
    return n < 63 ? n : 63;  // the counter holds six bits
}

}  // namespace dvi

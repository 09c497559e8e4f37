// Order of the exchanges between the two waves of a marching strip
// (step_march.hpp), in plain C++.
//
// An exchange: each wave writes its half of a buffer, both meet at one barrier,
// both read the two halves.  Nothing but that barrier orders the waves, so a
// wave may write its half for the next exchange while the other has not read
// this one's yet.  Two buffers that alternate make that safe: the write that
// reuses a buffer comes two exchanges later, behind the barrier of the exchange
// between, which the other wave reaches only after it has read.  So no two
// exchanges in a row may use the same buffer.
#pragma once

namespace cdbm {

// A piece's iterations, counted from its first row less four: the first four
// move the state of stage 1 only, the next four run stage 1, the rest both
// stages (the last of them may run stage 1 only).
constexpr int MARCH_TAKE = 4, MARCH_ONE = 4;

// The buffer of the exchange of `stage` (0 or 1) in an iteration.
constexpr int march_buffer(int iteration, int stage) {
    return iteration < MARCH_TAKE + MARCH_ONE ? iteration & 1 : stage;
}

// The exchanges of stage 1 alone alternate, and the first iteration of both
// stages starts with the buffer that the last of them left.
static_assert(march_buffer(MARCH_TAKE + MARCH_ONE - 1, 0) != march_buffer(MARCH_TAKE + MARCH_ONE, 0) &&
                  march_buffer(MARCH_TAKE + MARCH_ONE, 0) != march_buffer(MARCH_TAKE + MARCH_ONE, 1),
              "no two exchanges in a row through one buffer");

}  // namespace cdbm

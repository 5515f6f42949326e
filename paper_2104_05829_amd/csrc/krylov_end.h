// How the launches of a Krylov iteration learn that a vector's iteration has ended.
#pragma once

namespace semx {

// Launches of iteration `it` that may end it.  A flexible CG uses the update, the
// convergence test and the direction, Jacobi-PCG the operator (which decides on the
// iteration before), the update and the decision at a batch's end.
enum KrylovLaunch { kEndOperator = 0, kEndUpdate = 1, kEndDecide = 2, kEndDirection = 3 };

// The launch's stamp: neither 0 (running) nor 1 (ended at the start), and another
// one than that of every launch enqueued near it.
constexpr int end_stamp(int it, KrylovLaunch k)
{
    return 0x40000000 | (int)((3LL * it + k) & 0x3fffffff);
}

// Whether a launch has nothing to do.  `done` is 0 until one block of the launch
// that ends the iteration writes that launch's stamp.  Blocks of the same launch
// read the flag on either side of the write, wavefronts of one block too, and then
// meet at barriers: an own stamp counts as 0, so that they go the same way, and
// each takes the decision that led to the write from the same sums.
constexpr bool ended_before(int done, int stamp) { return done != 0 && done != stamp; }

}  // namespace semx

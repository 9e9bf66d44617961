// How many of a wavefront's copies may still be under way when a chunk of linear_pipe.hip ends (host and device code).
//
// A chunk's copies are `near` ones, for the chunk three further on (activations, group scales), and `far` ones, for the chunk four further
// on (nibbles, records).  What the next chunk reads was issued before this chunk's copies, so the wait at its end leaves those under way
// and nothing else.  Behind the end of K they are copies of no lanes.  A load takes its place in the count behind the older ones, but
// whether one without lanes does is not said anywhere: if it took none, a wait for all but the usual number would let a
// wavefront read what has not arrived.  So they do not count as left.
#pragma once

namespace w4a8 {

// left: chunks from the one that ends on, itself included
constexpr int copies_that_may_be_left(int near, int far, int left) { return (left > 3 ? near : 0) + (left > 4 ? far : 0); }

}  // namespace w4a8

// How far the sweeps with a sparse part read behind the stored values, in plain C++ so that it can be checked on a host.
#pragma once

namespace lcn {

// A sweep requests the first chunks (64 entries, a wavefront's worth) of a row's record together with the row, and the
// rest of a longer record in trips of several chunks.  No lane of these loads is predicated: what lies past the record's end
// is read and masked when it is used.
constexpr int SWEEP_TRIP = 6;   // chunks of a trip, rows of up to 256 factor entries (pass_kernel)
constexpr int LONG_TRIP = 4;    // ... and longer ones (long_pass_kernel)

// Entries read past the end of a record of `total` entries, `first` chunks of it with its row, the rest in trips.
constexpr int read_past_end(int total, int first, int trip)
{
    int end = 64 * first;
    while (end < total) end += 64 * trip;
    return end > total ? end - total : 0;
}

// Floats behind the stored values that a sweep may read.  A trip starts inside the record, so less than a whole one of
// it lies outside; a record without entries is read for its first chunks (each kernel asserts both).
constexpr int VALUE_SLACK = 64 * (SWEEP_TRIP > LONG_TRIP ? SWEEP_TRIP : LONG_TRIP);

}  // namespace lcn

// Tickets of a launch that combines its own records (attend.hip): one 32-bit word per query head, to which
// the writer of each of the head's P records adds its step once the record is stored; the step that brings the
// word to zero is the last one, and its writer combines the records.
//
// The steps of a head's records add up to zero (modulo 2^32) and no smaller set of them does: record 0 steps
// back by P - 1, every other one steps forward by 1. So the word is zero again as soon as every launch that
// was started has run to its end, in whatever order their steps were taken and however many records each had.
// Nothing has to clear it, and calls that overlapped (whose own results are undefined: they share the
// records) leave nothing behind for later ones. A count that the last writer sets back to zero does not have
// that property: two overlapping calls can leave it off, and then no later call ever finds its last record.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define RA_HOST_DEVICE __host__ __device__
#else
#define RA_HOST_DEVICE
#endif

RA_HOST_DEVICE static inline uint32_t ticket_step(int record, int records) {
    return record == 0 ? 1u - (uint32_t)records : 1u;
}
// `before`: the word as the atomic addition of `step` found it
RA_HOST_DEVICE static inline bool ticket_last(uint32_t before, uint32_t step) { return before + step == 0u; }

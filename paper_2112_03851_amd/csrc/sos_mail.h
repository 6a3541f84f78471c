// Sequence numbers of the on-chip form's mailboxes (sos_chip.h): plain C++, so
// that a host program can run the protocol through every order of its steps.
#pragma once

#include <stdint.h>

namespace sos {

// A team member writes w of its edge planes into mailboxes that its neighbour
// reads, two of each, used in turn (the parity of the sequence number). It may
// write sweep k + 2 over sweep k once its neighbour has read k, which it knows from
// the meeting of sweep k + 1: a member publishes its sums there only after it has
// read k. So the sweeps of a team are numbered without a gap, from one subdomain
// to the next too: a subdomain that needs no sweep (r_s already meets the
// tolerance, or is zero) has no meeting, and must not move the parity on.
constexpr uint32_t mail_next_job(uint32_t last_sweep) { return last_sweep + 1; }

}  // namespace sos

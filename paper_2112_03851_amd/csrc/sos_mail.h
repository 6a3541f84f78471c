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

// A mailbox word counts as sent when it carries the number of the sweep, so no
// other word there may carry it: not 0, which cleared words hold, and none that an
// earlier sweep used since the mailboxes were cleared (a slot that few subdomains
// reach keeps its words for many launches). Each launch has numbers of its own,
// as many as a team can need: one subdomain and every one that the other teams
// leave, max_inner + 1 sweeps each (at most 2^31 sweeps, which take hours). When
// they are used up the host clears the mailboxes and the launch count.
constexpr uint32_t mail_span(int64_t n_jobs, int64_t n_teams, int64_t max_inner) {
  const int64_t jobs = n_jobs > n_teams ? n_jobs - n_teams + 1 : 1;
  const int64_t most = int64_t(1) << 31;
  return uint32_t(max_inner >= most / jobs ? most : jobs * (max_inner + 1));
}
// Launches between two clears.
constexpr uint32_t mail_launches(uint32_t span) { return UINT32_MAX / span; }
// The first number of a launch, counted from 1 since the last clear.
constexpr uint32_t mail_first(uint32_t launch, uint32_t span) { return (launch - 1) * span + 1; }

}  // namespace sos

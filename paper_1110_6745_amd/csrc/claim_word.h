// The claim words of the persistent batch kernel: (sweep << 32) | low word.  Plain
// constexpr functions, so that the same rules are built into the kernel and into
// CPU checks.
#pragma once

#include <cstdint>

namespace okpz {
namespace batch {

// claim[r] = (sweep << 32) | next item to hand out; job r has an open item
// while the low word is below nitems[r] (its items per sweep).  A finished or empty job holds
// kClosed in the low word.  A scan can see a word open that is exhausted or
// closed by the time the wave's fetch-and-add lands, and a workgroup tries the job
// of its previous claim without a look (kClaimSticky); such late increments are
// at most two claims of two items per workgroup and word value, as a workgroup that
// finds nothing prefers no job (preferred_job).  So the low word never carries into
// the sweep number (kClosed + 4 * 2^16 < 2^32).  A job
// advanced by a team (kClaimStay) holds kTeam: nothing to claim, but its members go on.
constexpr uint32_t kClosed = 0x80000000u, kTeam = 0x40000000u;

// Whether a workgroup that waits for sweep s of a job goes on with its team, from a claim
// word that is no longer of sweep s.  The team of s + 1 cannot finish that sweep
// without every member, so a member never sees a later one; a waiter whose sweep
// did not become a team may find that others have formed one since.
constexpr bool team_goes_on(uint64_t word, uint32_t s)
{
    return (uint32_t)(word >> 32) == s + 1 && (uint32_t)word >= kTeam && (uint32_t)word < kClosed;
}

// The job that a workgroup tries first at its next look, after one that claimed items
// of job `claimed` (-1: nothing was open anywhere): that job, or none.  Trying the last
// job again after a look that found nothing would add to its closed word at every look,
// without bound, and reopen the finished job once the low word is full (hundreds of
// workgroups beside one long job: a minute or two).
constexpr int preferred_job(int claimed) { return claimed; }

}  // namespace batch
}  // namespace okpz

// CPU check of the batch kernel's claim-word rules (csrc/claim_word.h): who goes on
// as a team after a sweep, and what looks for work add to a word.  Prints "claim words
// ok" or the first fault.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "claim_word.h"

using namespace okpz::batch;

static void require(bool ok, const char *what)
{
    if (!ok) {
        std::printf("%s\n", what);
        std::exit(1);
    }
}

static uint64_t word(uint32_t sweep, uint32_t low) { return (uint64_t)sweep << 32 | low; }

int main()
{
    // A workgroup that has completed items of sweep s and waits for it sees the word
    // change to one of: s + 1 as a team, s + 1 open, s + 1 closed, or, having looked
    // away meanwhile, any later state of a job that other workgroups advance.
    for (uint32_t s : {0u, 1u, 77u, 0x7ffffffdu}) {
        for (uint32_t late = 0; late <= 1024; late += 256) {  // late increments
            require(team_goes_on(word(s + 1, kTeam + late), s), "the team of sweep s does not go on");
            require(!team_goes_on(word(s + 1, late), s), "an open sweep taken for a team");
            require(!team_goes_on(word(s + 1, kClosed + late), s), "a closed job taken for a team");
            for (uint32_t ahead : {2u, 3u, 100u})
                for (uint32_t low : {0u, kTeam, kClosed})
                    require(!team_goes_on(word(s + ahead, low + late), s), "a later team taken for the sweep's own");
        }
    }
    // The schedule that needs it: W waits for sweep 0, which did not become a team;
    // others claim and complete sweep 1, form a team there, and only then W looks.
    {
        const uint32_t nitems = 4;
        uint64_t w = word(0, nitems);          // every item of sweep 0 handed out
        w = word(1, 0);                        // completed without a team: open again
        for (uint32_t i = 0; i < nitems; ++i) ++w;
        w = word(2, kTeam);                    // completed by workgroups that all stayed
        require(!team_goes_on(w, 0), "a waiter of sweep 0 joins the team of sweep 2");
    }
    // Workgroups that look on for work after their job's end, while one other job
    // still runs: the closed word must not creep towards the next sweep's number.
    {
        const int job = 3, looks = 100000, workgroups = 512;
        uint64_t w = word(40, kClosed);
        for (int g = 0; g < workgroups; ++g) {
            int prefer = job;  // claimed from it last
            for (int i = 0; i < looks; ++i) {
                if (prefer >= 0) w += 2;  // the try of two items without a look
                prefer = preferred_job(-1);
            }
        }
        require(w >> 32 == 40 && (uint32_t)w >= kClosed, "looks for work reopen a finished job");
        require((uint32_t)w - kClosed <= 2u * workgroups, "looks for work add to a closed word without bound");
    }
    require(preferred_job(5) == 5 && preferred_job(0) == 0, "the previous claim's job is not preferred");
    std::printf("claim words ok\n");
    return 0;
}

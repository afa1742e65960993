// Hooks for the library's own tests, not part of the public headers.
#pragma once

#include "../../include/tns_cache.h"

// Test of what a cache update does when the tiles of its chained scan do not hear from one another: no tile of this
// cache's updates waits for those before it, as after a bounded wait that ran out.
extern "C" TNS_API void tns_test_cache_no_wait(tns_cache* cache);

// Accepted in tns_config.flags.  Test of the fused kernel's bounded wait: the tiles start at 1, so the first tile's predecessor
// never reports.  Every kernel still ends (with tickets after the bound, about two seconds; without, where the missing tile has not
// said that it started, after two milliseconds); tns_run_status then reports the time-out and the dense outputs are not valid.
#define TNS_TEST_FLAG_LOST_TILE 64

// Batches without tickets: from now on a tile of this plan's calls that does not find the totals before it at its first look makes
// room, also where the missing tiles have started.  The results are what they always are.  The 64-bit word at byte 8 of the
// workspace counts the tiles that were sampled again.
extern "C" TNS_API void tns_test_defer(tns_plan* plan);

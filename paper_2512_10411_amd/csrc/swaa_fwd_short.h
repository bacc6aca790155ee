// Forward of short prompts, head dimension 128 (swaa_fwd_short.hip): parameter block, dispatch rule and launcher.
#ifndef SWAA_FWD_SHORT_H_
#define SWAA_FWD_SHORT_H_

#include "swaa_common.h"

namespace swaa {

struct FwdShortParams {
    FwdParams f;
    int pairs, tiles;            // (batch, KV head) pairs; 32-row tiles of a sequence
    FastDiv div_pairs, div_group;  // pairs and f.G
};

// Does the call (planned, keys whole) run on the short prompts' kernel?  Fills sp if so.
bool plan_fwd_short(const FwdParams &p, FwdShortParams &sp);
hipError_t launch_fwd_short_d128(const FwdShortParams &sp, hipStream_t stream);

}  // namespace swaa

#endif  // SWAA_FWD_SHORT_H_

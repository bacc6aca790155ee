// Forward of short prompts: parameter block, and the dispatch rule and launcher of head dimension 128 (swaa_fwd_short.hip).
#ifndef SWAA_FWD_SHORT_H_
#define SWAA_FWD_SHORT_H_

#include "swaa_common.h"

namespace swaa {

struct FwdShortParams {
    FwdParams f;
    int pairs, tiles;            // (batch, KV head) pairs; 32-row tiles of a sequence
    FastDiv div_pairs, div_group;  // pairs and f.G
};

// Fills sp for the call p, in units of 32 rows of a head.
inline void fill_fwd_short(const FwdParams &p, FwdShortParams &sp) {
    sp.f = p;
    sp.pairs = p.B * p.Hkv;
    sp.tiles = (p.Nq + 31) / 32;
    sp.div_pairs = make_fastdiv((unsigned)sp.pairs);
    sp.div_group = make_fastdiv((unsigned)p.G);
}

// Does the call (planned, keys whole) run on the short prompts' kernel?  Fills sp if so.  general: a call of the general form.
bool plan_fwd_short(const FwdParams &p, bool general, FwdShortParams &sp);
hipError_t launch_fwd_short_d128(const FwdShortParams &sp, hipStream_t stream);

}  // namespace swaa

#endif  // SWAA_FWD_SHORT_H_

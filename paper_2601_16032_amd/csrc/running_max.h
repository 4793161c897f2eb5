// The lazily raised reference maximum of the online softmax, for kernels that compare raw scores with a limit instead of
// shifted ones with a slack (host code can include this too).
//
// A row's scores are taken relative to M = t * c, t the raw maximum of an earlier tile and c = |scale| * log2(e).  M is
// raised only for a score above score_limit(): up to there probabilities are at most 2^kRescaleSlack (a factor that O and
// the running sum share, so the result is unchanged), and rescaling the accumulators on almost every tile is saved.
#pragma once

#include <math.h>

#include "schedule.h"      // SAW_HD

namespace sawattn {

constexpr float kRescaleSlack = 8.0f;

// Raw score above which a reference M = t * c has to be raised.  The limit keeps a distance of |M| 2^-21 from M + slack,
// which covers the rounding of the division and of the comparison on raw scores.  It never lies below t itself: beyond
// |M| = 2^24 the distance is larger than the slack, and a limit below t would let a smaller maximum than the present one
// lower the reference -- O and the running sum would grow by a power of two each time, without bound.  (fmaxf also
// ignores the NaN of an infinite M: then only a larger score, that is none, asks for another raise.)
SAW_HD float score_limit(float t, float M, float c) {
    return fmaxf(t, (M + kRescaleSlack - fabsf(M) * 0x1p-21f) / c);
}

}  // namespace sawattn

// lds_bucket.h -- the buckets of the in-LDS sort (tree_build.hip).  Plain C++ as well,
// so that the rule is tested on the CPU (tests/test_lds_bucket.py).
#pragma once

#include <cmath>

#ifdef __HIP__
#define FMM_BUCKET_FN __host__ __device__ __forceinline__
#else
#define FMM_BUCKET_FN inline
#endif

namespace fmm {

// bucket of a coordinate among nb of equal width from lo on (scale: buckets per
// unit) and the place inside it, 0 .. 1; monotone in the coordinate.  The largest
// coordinate lies at the end of the last bucket (place 1).
struct LdsPlace {
    int bucket;
    double place;
};
FMM_BUCKET_FN LdsPlace lds_place(double c, double lo, double scale, int nb)
{
    const double v = fmin(fmax((c - lo) * scale, 0.0), (double)nb);
    const int b = (int)v < nb - 1 ? (int)v : nb - 1;
    return LdsPlace{b, v - (double)b};
}

// the second level: a bucket whose points take the places first .. end - 1 becomes
// that many buckets of equal width
FMM_BUCKET_FN int lds_finer(double place, int first, int end)
{
    const int n = end - first, k = (int)(place * (double)n);
    return first + (k < n - 1 ? k : n - 1);
}

}  // namespace fmm

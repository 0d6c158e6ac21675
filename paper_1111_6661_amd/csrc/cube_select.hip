// cube_select.hip -- exact selection (k-th smallest valid voxel) and the
// median: the global, multi-pass median task the paper names in Section 3.
// One or two ranks of the order statistics: a large box is read once
// (cube_bracket.h); otherwise the passes of cube_quantile.hip read it twice,
// and the voxels of the wanted leading key buckets a third time.
#include "cube_internal.h"

using namespace cube;

extern "C" {

int cube_select(const float *ptr, const int64_t *dims, uint64_t rank, float *value)
{
    CUBE_GUARD_BEGIN
    if (!value) return fail(CUBE_EINVAL, "value is NULL");
    Box b;
    int rc = check_box(ptr, dims, &b);
    if (!rc) rc = check_box_device(&b);
    if (rc) return rc;
    if (b.n == 0) return fail(CUBE_EINVAL, "empty box");
    float v[2];
    int n_v = 0;
    uint64_t n = 0;
    if ((rc = box_ranks(b, 0, rank, v, &n_v, &n))) return rc;
    *value = v[0];
    return CUBE_OK;
    CUBE_GUARD_END
}

int cube_median(const float *ptr, const int64_t *dims, double *median, uint64_t *n_valid)
{
    CUBE_GUARD_BEGIN
    if (!median) return fail(CUBE_EINVAL, "median is NULL");
    Box b;
    int rc = check_box(ptr, dims, &b);
    if (!rc) rc = check_box_device(&b);
    if (rc) return rc;
    if (b.n == 0) return fail(CUBE_EINVAL, "empty box");
    // The lower middle (which is the median for odd n_valid) and, for even
    // n_valid, the upper middle too.
    float v[2];
    int n_v = 0;
    uint64_t n = 0;
    rc = box_ranks(b, 1, 0, v, &n_v, &n);
    if (n_valid) *n_valid = n;
    if (rc) return rc;
    *median = n_v == 1 ? (double)v[0] : ((double)v[0] + (double)v[1]) / 2.0;
    return CUBE_OK;
    CUBE_GUARD_END
}

}  // extern "C"

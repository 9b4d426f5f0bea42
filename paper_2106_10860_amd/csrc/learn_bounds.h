// How far the learner's estimates and the sums that they stand for can be apart.  What comes out of a level is a column and
// its thresholds, whole choices: the largest of some losses, the least of others.  Sums in any order, of which there is no
// chain, name the same one as the sums in Algorithms 3 and 4's order wherever the next best is further away than both can be
// off; where it is not, the exact sums tell.  With u = 2^-53, n rows and S the sum of the squares of a bucket's values, over all
// columns where several are summed, a chain of n additions is off by n u of the sum of its terms' sizes at most, one of h by
// h u, and sums over rows are at most sqrt(n S) (Cauchy-Schwarz).
#pragma once

namespace maddness {

// L(j, B).  As the exact kernel computes it: the mean is off by (n + 2) u sum|x| / n, which adds n times its square to the
// loss, and the sum of squares by (n + 3) u of itself.  As sum y^2 - (sum y)^2 / n with y = x - p for a p among the values:
// (3 n + 12) u sum y^2.  Together less than (4 n + 16) u Sy + (n + 2)^2 2^-104 (Sy + n p^2), the sum over the
// buckets 16 u Sy more; loss_error is twice that.  (0 for a column of zeros, whose loss is 0 either way.)
constexpr double loss_error(double n, double sy, double p)
{
    return (8.0 * n + 64.0) * 0x1p-53 * sy + (n + 2.0) * (n + 2.0) * 0x1p-103 * (sy + n * p * p);
}

// The loss of a bucket's split, or of the bucket where it has none.  In Algorithm 4's order a column's two halves are off by
// (3 n + 4) u of their squares' sum, their sum over d columns by d + 2 of it more; L(B), which takes their place where a candidate
// cannot split the bucket, by (n + d + 4) u S.  The estimate is a constant less the gain  sum_j w_j^2 n / (n1 n2),
// w_j = s_j - n1 T_j / n, from sums s_j, T_j that are off by h u sum|x| with h <= 256 + N / 2^18 (32 rows, 8 tiles, the scan of the
// groups; N: rows of all buckets): |w_j| n / (n1 n2) is at most 2 sqrt(S_j), so the gain is off by 8 h sqrt(n) u S, and some 100 u S
// for its products and sums.  exact_sums: all sums of values and of their squares are exact in any order, which leaves d + 8 and
// 16 sqrt(n) of the splits.  L(B) sums squares of what is left of the mean, which are not exact: binary values in 2^20
// rows leave it off by 180000 u S, where 64 sqrt(n) is 65536.  So its n + d + 4 stay unless every candidate splits the bucket.
// root: sqrt(n); rows: N; energy: S.
constexpr double split_error(double n, double root, double rows, double energy, int d, bool exact_sums, bool every_splits)
{
    const double units = !exact_sums ? 8.0 * n + 8.0 * (256.0 + rows * 0x1p-18) * root : every_splits ? 64.0 * root : 64.0 * root + 4.0 * n;
    return (units + 16.0 * d + 1024.0) * 0x1p-53 * energy;
}

}  // namespace maddness

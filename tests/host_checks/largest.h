// The largest error so far.  A NaN counts as larger than any number and stays: std::max and std::fmax pass over it, so that
// a transform with a NaN among its results would look exact.
#pragma once
template <class T> inline void keep_largest(T &worst, T error)
{
    if (error > worst || error != error) worst = error;
}

// Grouping of a long list by a bucket key on the device (lm_sort.hip): the
// counting sort that orders events by transaxial line for the forward
// projection by line.
#pragma once

#include <hip/hip_runtime.h>

namespace lmk {

// Largest number of buckets group_by_key handles (two digits of 9 bits).
constexpr unsigned kGroupMaxBuckets = 1u << 18;

// out[off[b] .. off[b + 1]) = the indices of the elements with key b, for
// every bucket b < nb (their order inside a bucket is not fixed); elements
// with key >= nb are dropped; off has nb + 1 entries.  n < 2^31, nb <=
// kGroupMaxBuckets.  Two passes of per-workgroup counting in LDS, one per
// 9-bit digit of the key (most significant first), each reserving its
// ranges with one global atomic per workgroup and digit value instead of one
// per element.  Temporaries are allocated and freed stream-ordered;
// LM_ENOMEM when they do not fit (nothing enqueued).
int group_by_key(const unsigned *key, long long n, unsigned nb, unsigned *out, unsigned *off, hipStream_t st);

}  // namespace lmk

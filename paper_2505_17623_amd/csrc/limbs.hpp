// limbs.hpp -- sums of eq values times small integers.  An eq value is cut into
// limbs whose products with the entries are exact multiply-adds into int64 over
// a bounded run of entries; each run is reduced mod p once.  (A product reduced
// per entry costs about 25 instructions, a limb's multiply-add one.)
#pragma once
#include "m61.hpp"

namespace ra {

template <typename T> struct BindLimbs;
template <> struct BindLimbs<int16_t> {
    static constexpr int kBits = 31, kCount = 2, kRun = 1 << 15;  // |limb entry| < 2^46: 2^15 terms below 2^61
};
template <> struct BindLimbs<int32_t> {
    static constexpr int kBits = 21, kCount = 3, kRun = 1 << 9;  // 2^52
};
// the element a limb sum stands for
template <int BITS, int CNT> __device__ __forceinline__ uint64_t limbs_value(const int64_t (&a)[CNT])
{
    uint64_t v = 0;
#pragma unroll
    for (int i = 0; i < CNT; i++) v = m61::add(v, m61::rotl(m61::from_i64(a[i]), BITS * i));
    return v;
}

}  // namespace ra

// 64-bit sums that may wrap.
#pragma once

#include <cstdint>

namespace mm {
namespace dev {

// a b + t mod 2^64 (one 64-bit multiply-add).  The sums that carry a bias of 2^63 and more, so
// that a reduction ends in balanced bytes, leave int64_t on ordinary values.
constexpr int64_t mad_wrap(int32_t a, int32_t b, int64_t t)
{
    return (int64_t)((uint64_t)((int64_t)a * b) + (uint64_t)t);
}

}  // namespace dev
}  // namespace mm

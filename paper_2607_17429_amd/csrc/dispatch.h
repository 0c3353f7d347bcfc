// Compile-time dispatch of the orbit-search kernels over the label word (labels
// of up to 32 bits are searched in uint32_t) and the candidate-set words.
#pragma once

#include <cstdint>
#include <type_traits>

namespace ftlm {

// label word of the H.V kernels' chunk-count parameter (8: 32 bits, 16: 64 bits)
template <int NCH>
using word_t = typename std::conditional<(NCH <= 8), uint32_t, uint64_t>::type;

// 64-bit words of a candidate set over a group of `order` elements (dev::Orbit)
inline int orbit_words(int order) { return order <= 128 ? 2 : order <= 320 ? 5 : order <= 1024 ? 16 : -1; }

#define FTLM_ORBIT_CASE(n, T, P, ...)     \
  case n: {                               \
    using W = T;                          \
    constexpr int GW = n;                 \
    constexpr bool PLAIN = P;             \
    __VA_ARGS__;                          \
  } break;

#define FTLM_ORBIT_CASES(T, P, gw, ...)                                                           \
  switch (gw) {                                                                                   \
    FTLM_ORBIT_CASE(2, T, P, __VA_ARGS__) FTLM_ORBIT_CASE(5, T, P, __VA_ARGS__)                   \
    FTLM_ORBIT_CASE(16, T, P, __VA_ARGS__)                                                        \
    default: ::ftlm::fail(FTLM_ERR_GROUP_TOO_LARGE, "group order above 1024");                    \
  }

#define FTLM_DISPATCH_ORBIT(wide, plain, gw, ...)                                                 \
  if (wide) {                                                                                     \
    if (plain) {                                                                                  \
      FTLM_ORBIT_CASES(uint64_t, true, gw, __VA_ARGS__)                                           \
    } else {                                                                                      \
      FTLM_ORBIT_CASES(uint64_t, false, gw, __VA_ARGS__)                                          \
    }                                                                                             \
  } else {                                                                                        \
    if (plain) {                                                                                  \
      FTLM_ORBIT_CASES(uint32_t, true, gw, __VA_ARGS__)                                           \
    } else {                                                                                      \
      FTLM_ORBIT_CASES(uint32_t, false, gw, __VA_ARGS__)                                          \
    }                                                                                             \
  }

}  // namespace ftlm

// What the traversal and dealing headers take from the HIP runtime, for the lane emulation in lanes.cpp:
// the lanes run as coroutines, and an exchange between lanes returns only when all of them have come
// to the same one.  Lanes at different exchanges, or some of them finished, are a fault of the code.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

using std::max;
using std::min;

#define __host__
#define __device__
#define __forceinline__ inline __attribute__((always_inline))
#define __restrict__ __restrict

struct float3 { float x, y, z; };
struct float4 { float x, y, z, w; };
inline float3 make_float3(float x, float y, float z) { return {x, y, z}; }

namespace lanes {
int current();                                           // the running lane
uint64_t exchange(int site, uint64_t v, int from);       // v of lane `from`; -1: bit i is v of lane i
uint64_t counter_read(const unsigned long long* c);      // other waves move the counter between any two accesses
uint64_t counter_add(unsigned long long* c, unsigned long long n);
template <class T> T exchange_as(int site, T v, int from) {
    uint64_t u = 0;
    std::memcpy(&u, &v, sizeof(T));
    u = exchange(site, u, from);
    std::memcpy(&v, &u, sizeof(T));
    return v;
}
}  // namespace lanes

#define __shfl_xor(v, o) lanes::exchange_as(__COUNTER__, v, lanes::current() ^ (o))
#define __shfl(v, from) lanes::exchange_as(__COUNTER__, v, from)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(c, order, scope) lanes::counter_read(c)
inline unsigned long long atomicAdd(unsigned long long* c, unsigned long long n) { return lanes::counter_add(c, n); }
inline int __lane_id() { return lanes::current(); }
inline int __popcll(uint64_t m) { return __builtin_popcountll(m); }
inline uint64_t __ballot(bool p) { return lanes::exchange(-2, p, -1); }

// Stand-in for the runtime header with which g++ compiles the device functions
// of af_device.h, sixteen threads of the host as the lanes of a group.  Test
// infrastructure.
#pragma once
#include <atomic>
#include <barrier>
#include <cmath>
#include <cstdint>
#include <cstring>
using std::exp;
using std::fabs;
using std::fma;
using std::fmax;
using std::fmin;
using std::ldexp;

#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / std::sqrt(x))
#define __builtin_amdgcn_sqrtf(x) std::sqrt((float)(x))
#define __expf(x) std::exp((float)(x))

inline unsigned long long atomicAdd(unsigned long long* p, unsigned long long v) {
  return __atomic_fetch_add(p, v, __ATOMIC_RELAXED);
}
inline void atomicMax(unsigned long long* p, unsigned long long v) {
  unsigned long long q = __atomic_load_n(p, __ATOMIC_RELAXED);
  while (q < v && !__atomic_compare_exchange_n(p, &q, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {}
}
inline void atomicMin(unsigned long long* p, unsigned long long v) {
  unsigned long long q = __atomic_load_n(p, __ATOMIC_RELAXED);
  while (q > v && !__atomic_compare_exchange_n(p, &q, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {}
}
inline long long __double_as_longlong(double x) {
  long long r;
  std::memcpy(&r, &x, 8);
  return r;
}

// The lanes of one group: each call is met by all of them.
constexpr int LANES = 16;
inline std::barrier<> lane_barrier(LANES);
inline double lane_value[LANES];
inline thread_local int lane_id;
inline double __shfl_xor(double v, int m) {
  lane_value[lane_id] = v;
  lane_barrier.arrive_and_wait();
  const double r = lane_value[lane_id ^ m];
  lane_barrier.arrive_and_wait();
  return r;
}
inline unsigned long long __ballot(bool p) {
  lane_value[lane_id] = p;
  lane_barrier.arrive_and_wait();
  unsigned long long r = 0;
  for (int k = 0; k < LANES; ++k) r |= (unsigned long long)(lane_value[k] != 0.0) << k;
  lane_barrier.arrive_and_wait();
  return r;
}

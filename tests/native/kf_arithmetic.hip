// Device checks of the fit's short arithmetic (tpcca_kf.h) against the
// correctly rounded operations.  Each entry point runs its checks on the
// current device and returns how many it made and how many differed.
#include "tpcca_kf.h"

namespace {

using u64 = unsigned long long;

struct Count {
  u64 done, wrong;
};

__device__ bool same(float a, float b) {
  return __float_as_uint(a) == __float_as_uint(b) || (a != a && b != b);
}

// A thread's totals.
__device__ void add(Count *c, unsigned int done, unsigned int wrong) {
  atomicAdd(&c->done, (u64)done);
  if (wrong) atomicAdd(&c->wrong, (u64)wrong);
}

__device__ float of(int e, unsigned int m) { return __uint_as_float(((unsigned int)(127 + e) << 23) | (m & 0x7FFFFFu)); }

__global__ void k_reciprocal(Count *c) {
  const unsigned int m = blockIdx.x * blockDim.x + threadIdx.x;
  unsigned int done = 0, wrong = 0;
  for (int e = -122; e <= 122; ++e, ++done) {
    const float d = of(e, m), want = 1.0f / d;
    const tpcca::KRecip r = tpcca::kf_recip(d);
    wrong += !same(r.r, want) || !same(tpcca::kf_div(1.0f, r), want);
  }
  add(c, done, wrong);
}

// every float bit pattern: 256 to a thread
__global__ void k_inverse(Count *c) {
  const unsigned int i0 = (blockIdx.x * blockDim.x + threadIdx.x) << 8;
  unsigned int done = 0, wrong = 0;
  for (unsigned int k = 0; k < 256; ++k, ++done) {
    const float d = __uint_as_float(i0 + k), want = 1.0f / d;
    // alone in its wave's vote and beside the other lanes
    float alone = tpcca::kf_div(1.0f, tpcca::kf_recip(d));
    if (!__builtin_amdgcn_classf(alone, 0x108)) alone = 1.0f / d;
    wrong += !same(alone, want) || !same(tpcca::kf_inverse(d), want);
  }
  add(c, done, wrong);
}

__global__ void k_root(Count *c) {
  const unsigned int m = blockIdx.x * blockDim.x + threadIdx.x;
  unsigned int done = 0, wrong = 0;
  for (int e = -96; e <= 120; ++e, ++done) wrong += !same(tpcca::kf_sqrt(of(e, m)), sqrtf(of(e, m)));
  add(c, done, wrong);
}

__device__ unsigned int next(u64 &s) {
  s = s * 6364136223846793005ull + 1442695040888963407ull;
  unsigned int x = (unsigned int)((s >> 33) ^ (s >> 18));
  x ^= x >> 15;
  x *= 0x2C1B3C6Du;
  return x ^ (x >> 12);
}

__global__ void k_quotient(Count *c, int per) {
  u64 s = 0x9E3779B97F4A7C15ull * (blockIdx.x * blockDim.x + threadIdx.x + 1);
  unsigned int wrong = 0;
  for (int k = 0; k < per; ++k) {
    unsigned int a = next(s), b = next(s);
    const unsigned int m = next(s);
    // significands that begin with ones or zeros, where quotients come close to a tie
    if ((m & 15) == 0) a |= 0x7FFF00u;
    if ((m & 0xF0) == 0) b |= 0x7FFF00u;
    if ((m & 0xF00) == 0) a &= ~0x7FFF00u;
    if ((m & 0xF000) == 0) b &= ~0x7FFF00u;
    const float n = of((int)((m >> 16) % 61) - 30, a) * (a >> 31 ? -1.0f : 1.0f);
    const float d = of((int)((m >> 24) % 61) - 30, b) * (b >> 31 ? -1.0f : 1.0f);
    wrong += !same(tpcca::kf_div(n, tpcca::kf_recip(d)), n / d);
  }
  add(c, per, wrong);
}

__global__ void k_special(Count *c) {
  const float v[8] = {0.0f, -0.0f, 1.0f, -1.0f, __builtin_inff(), -__builtin_inff(), __builtin_nanf(""), 3.5f};
  const float n = v[threadIdx.x >> 3], d = v[threadIdx.x & 7];
  add(c, 1, !same(tpcca::kf_div(n, tpcca::kf_recip(d)), n / d));
  if (threadIdx.x < 8) add(c, 1, !same(tpcca::kf_sqrt(v[threadIdx.x]), sqrtf(v[threadIdx.x])));
}

template <class F>
int run(u64 *done, u64 *wrong, F &&launch) {
  Count *c = nullptr, h{};
  if (hipMalloc(&c, sizeof(Count)) != hipSuccess) return 1;
  hipError_t e = hipMemcpy(c, &h, sizeof(h), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    launch(c);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(&h, c, sizeof(h), hipMemcpyDeviceToHost);
  (void)hipFree(c);
  *done = h.done;
  *wrong = h.wrong;
  return e == hipSuccess ? 0 : 1;
}

}  // namespace

extern "C" {
int check_reciprocal(u64 *done, u64 *wrong) {
  return run(done, wrong, [](Count *c) { k_reciprocal<<<(1 << 23) / 256, 256>>>(c); });
}
int check_inverse(u64 *done, u64 *wrong) {
  return run(done, wrong, [](Count *c) { k_inverse<<<(1 << 24) / 256, 256>>>(c); });
}
int check_root(u64 *done, u64 *wrong) {
  return run(done, wrong, [](Count *c) { k_root<<<(1 << 23) / 256, 256>>>(c); });
}
int check_quotient(u64 *done, u64 *wrong) {
  return run(done, wrong, [](Count *c) { k_quotient<<<4096, 256>>>(c, 2048); });
}
int check_special(u64 *done, u64 *wrong) {
  return run(done, wrong, [](Count *c) { k_special<<<1, 64>>>(c); });
}
}

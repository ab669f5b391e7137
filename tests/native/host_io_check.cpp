// Checks of host_io.hpp against the runtime of hip/hip_runtime.h beside this
// file.  One argument: the check's name.  Exit status 0: it holds.
#include <chrono>
#include <cstdio>
#include <string>
#include <thread>
#include <vector>

#include "host_io.hpp"

using namespace epdlb;

#define REQUIRE(x)                                    \
  do {                                                \
    if (!(x)) {                                       \
      std::printf("line %d: %s\n", __LINE__, #x);     \
      return 1;                                       \
    }                                                 \
  } while (0)

namespace {

double value(size_t i, int seed) { return double((i * 2654435761u + unsigned(seed) * 40503u) % 16777213u); }

// The worker of the first chunk falls behind the others.
void slow(size_t i) {
  if (i == 0) std::this_thread::sleep_for(std::chrono::milliseconds(30));
}

template <typename T> hipError_t down(int device, MockStream& s, size_t count, int seed, bool* right) {
  std::vector<T> dev(count);
  for (size_t i = 0; i < count; ++i) dev[i] = T(value(i, seed));
  std::vector<double> out(count, -1.0);
  bool done = false;
  const hipError_t e = staged_download(device, &s, out.data(), dev.data(), count, [](size_t i, T v) { return slow(i), double(v); }, &done);
  *right = done;
  for (size_t i = 0; i < count && *right; ++i) *right = out[i] == value(i, seed);
  return e;
}
template <typename T> hipError_t up(int device, MockStream& s, size_t count, int seed, bool* right) {
  std::vector<double> src(count);
  for (size_t i = 0; i < count; ++i) src[i] = value(i, seed);
  std::vector<T> dev(count, T(-1));
  bool done = false, finite = false;
  const hipError_t e = staged_upload(device, &s, dev.data(), src.data(), count, [](size_t i, double v) { return slow(i), T(v); }, &finite, &done);
  *right = done && finite;
  for (size_t i = 0; i < count && *right; ++i) *right = dev[i] == T(value(i, seed));
  return e;
}

// A context's device is not the thread's current one.
int other_device_current() {
  StageUser a, b;
  MockStream s0, s1;
  s1.device = 1;
  const size_t n = 2 * kStageMin + 77;
  bool ok = false;
  hipSetDevice(1);
  REQUIRE(down<float>(0, s0, n, 1, &ok) == hipSuccess && ok);
  REQUIRE(mock().device == 1);
  REQUIRE(up<float>(0, s0, n, 2, &ok) == hipSuccess && ok);
  REQUIRE(down<float>(1, s1, n, 3, &ok) == hipSuccess && ok);
  hipSetDevice(0);
  REQUIRE(up<double>(1, s1, n, 4, &ok) == hipSuccess && ok);
  REQUIRE(down<double>(0, s0, n, 5, &ok) == hipSuccess && ok);
  REQUIRE(mock().device == 0 && mock().pins == 2);
  return 0;
}

// A transfer that fails gives its ring back to the system, not to the next one.
int failed_transfer() {
  StageUser a;
  MockStream s;
  bool ok = false;
  mock().fail_record = 3;
  REQUIRE(down<float>(0, s, 4 * kStageMin, 1, &ok) == hipErrorInvalidHandle);
  REQUIRE(mock().pins == 1 && mock().freed == 1);
  REQUIRE(down<float>(0, s, 4 * kStageMin, 2, &ok) == hipSuccess && ok);
  REQUIRE(mock().pins == 2 && mock().freed == 1);
  mock().fail_record = mock().records + 3;
  REQUIRE(up<float>(0, s, 4 * kStageMin, 1, &ok) == hipErrorInvalidHandle);
  REQUIRE(mock().freed == 2);
  REQUIRE(up<float>(0, s, 4 * kStageMin, 2, &ok) == hipSuccess && ok);
  REQUIRE(mock().pins == 3);
  return 0;
}

// FP64 planes and FP64 host arrays: below the ring's size the copies lie on the
// caller's array; values that change on the way (a type, an offset) do not.
int fp64_as_it_lies() {
  StageUser a;
  MockStream s;
  const size_t n = 98304;  // 3 planes of 64 x 32 x 16
  std::vector<double> src(n), dev(n, -1.0), out(n, -1.0);
  for (size_t i = 0; i < n; ++i) src[i] = value(i, 7);
  REQUIRE(host_upload(0, &s, dev.data(), src.data(), n, AsIs()) == hipSuccess);
  REQUIRE(mock().host == src.data() && dev == src);
  REQUIRE(host_download(0, &s, out.data(), static_cast<const double*>(dev.data()), n, AsIs()) == hipSuccess);
  REQUIRE(mock().host == out.data() && out == src && mock().copies == 2);
  REQUIRE(host_upload(0, &s, dev.data(), src.data(), n, [](size_t i, double v) { return v - double(i); }) == hipSuccess);
  REQUIRE(dev[0] == src[0] && dev[n - 1] == src[n - 1] - double(n - 1));
  REQUIRE(host_download(0, &s, out.data(), static_cast<const double*>(dev.data()), n,
                        [](size_t i, double v) { return v + double(i); }) == hipSuccess);
  REQUIRE(out == src);
  std::vector<float> f(n, -1.0f);
  REQUIRE(host_upload(0, &s, f.data(), src.data(), n, AsIs()) == hipSuccess);
  std::vector<double> back(n, -1.0);
  REQUIRE(host_download(0, &s, back.data(), static_cast<const float*>(f.data()), n, AsIs()) == hipSuccess);
  REQUIRE(back == src && mock().pins == 0);
  return 0;
}

// Every slot used several times, ragged and whole last chunks, the smallest sizes.
template <typename T> int over_the_ring() {
  StageUser a;
  MockStream s;
  const size_t ring = kStageSlotBytes / sizeof(T) * kStageSlots;
  bool ok = false;
  int seed = 0;
  for (size_t n : {size_t(1), kStageMin, kStageMin + 1, ring, ring + 1, 3 * ring, 3 * ring + ring / 3 + 5}) {
    REQUIRE(down<T>(0, s, n, ++seed, &ok) == hipSuccess && ok);
    REQUIRE(up<T>(0, s, n, ++seed, &ok) == hipSuccess && ok);
  }
  REQUIRE(mock().pins == 1);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "other_device_current") return other_device_current();
  if (what == "failed_transfer") return failed_transfer();
  if (what == "fp64_as_it_lies") return fp64_as_it_lies();
  if (what == "over_the_ring_fp32") return over_the_ring<float>();
  if (what == "over_the_ring_fp64") return over_the_ring<double>();
  std::printf("no check of that name\n");
  return 2;
}

// Host program: what is asked of the runtime once per device, with devices and answers of the test's own.
#include "../paper_2103_16063_amd/csrc/rannc_dp_once.h"

#include <cstdio>
#include <cstdlib>

int main() {
  std::atomic<uint64_t> done{0};
  int device = 0, asked[70] = {};
  hipError_t answer = hipSuccess;
  auto go = [&] {
    return rannc::once_per_device(done, [&](int *d) { *d = device; return device < 0 ? hipErrorNoDevice : hipSuccess; },
                                  [&] { ++asked[device]; return answer; });
  };
  const auto expect = [](bool ok, const char *what) {
    if (!ok) { std::printf("%s\n", what); std::exit(1); }
  };
  expect(go() == hipSuccess && go() == hipSuccess && asked[0] == 1, "once on a device");
  device = 1;
  expect(go() == hipSuccess && asked[1] == 1, "a second device is asked as well");
  device = 63;
  expect(go() == hipSuccess && go() == hipSuccess && asked[63] == 1, "the last device with a bit");
  device = 64;
  expect(go() == hipSuccess && go() == hipSuccess && asked[64] == 2, "devices without a bit are asked by every call");
  device = 2;
  answer = hipErrorInvalidValue;
  expect(go() == hipErrorInvalidValue, "a failure is reported");
  answer = hipSuccess;
  expect(go() == hipSuccess && asked[2] == 2, "a failure is not kept");
  device = -1;
  expect(go() == hipErrorNoDevice, "no current device");
  std::printf("ok\n");
  return 0;
}

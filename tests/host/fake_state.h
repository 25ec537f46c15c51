// What the test doubles of fake_hip.cpp record and are told.
#pragma once

#include <hip/hip_runtime.h>

#include <functional>
#include <map>
#include <string>
#include <vector>

namespace fake {

constexpr float kTable = 0.25f;   // every entry of a filled transform window

struct State {
  std::vector<float> strain;             // what the last ingest launch converted, when it ran
  std::function<void(const std::vector<float> &)> on_strain;   // the same, each time
  std::function<void()> before_sync;     // runs once, when a stream is next waited for: another thread's call
  float table = 0.f;                     // a transform window entry as the last conditioning launch saw it
  int64_t triggers = 0, pairs = 0;       // counts that the next calls report
  std::string fail_at;                   // call or launch that fails, once
  int fail_skip = 0;                     // how many calls of it succeed before
  std::map<std::string, int> calls;
};
extern State state;

void enqueue(hipStream_t s, std::function<void()> f);
size_t pending(hipStream_t s);
void drain(hipStream_t s);

}  // namespace fake

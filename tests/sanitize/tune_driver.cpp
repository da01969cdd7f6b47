// tune_driver.cpp -- the autotuner on the CPU: the planner and tuner linked
// against hip_host_stub.cpp, with an exec whose "time" is a rule on the tiles
// it would run on, so that which candidates are timed and which one stays is
// decided here and not by a clock.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <functional>
#include <string>
#include <vector>

#include "spinsum_plan_host.h"

namespace {
std::function<float(const spinsum_plan_s&)> g_time;
float g_ms = 0;
int g_failed = 0;

void check(bool ok, const std::string& what) {
  if (!ok) {
    std::printf("FAILED %s\n", what.c_str());
    ++g_failed;
  }
}
}  // namespace

// (hip_host_stub.cpp is compiled with its own versions of these renamed)
extern "C" hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
extern "C" hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
extern "C" hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = g_ms;
  return hipSuccess;
}
extern "C" spinsum_status spinsum_exec(spinsum_plan_t P, const void*, void*, void*) {
  g_ms = g_time(*P);
  return g_ms > 0 ? SPINSUM_OK : SPINSUM_ERR_UNSUPPORTED;
}

namespace {
struct Shape {
  const char* name;
  std::vector<int64_t> ext;
  int d;
  spinsum_dtype dtype;
  int inplace;
};

spinsum_plan_t make(const Shape& s) {
  // two terms that move every axis
  const int nterms = 2;
  std::vector<int> perms;
  for (int m = 0; m < s.d; ++m) perms.push_back(m);
  for (int m = 0; m < s.d; ++m) perms.push_back((m + 1) % s.d);
  const double alpha[2] = {1.0, -0.5};
  spinsum_plan_t p = nullptr;
  check(spinsum_plan(&p, (int)s.ext.size(), s.ext.data(), 1, s.d, 1, &nterms, perms.data(), alpha,
                     s.dtype, s.inplace, SPINSUM_FLAG_FULL_GROUP) == SPINSUM_OK,
        std::string(s.name) + ": plan");
  return p;
}

int lines(const std::string& path, std::string* last) {
  std::ifstream f(path);
  std::string l;
  int n = 0;
  while (std::getline(f, l)) {
    ++n;
    *last = l;
  }
  return n;
}

void run_case(const Shape& s, const std::string& dir) {
  const std::string path = dir + "/" + s.name;
  char buf[64];
  spinsum_plan_t p = make(s);
  spinsum_plan_info_t before, after;
  spinsum_plan_get_info(p, &before);
  check(before.sum_bl > 0 || before.persistent_per_cu > 0, std::string(s.name) + ": own kernel");
  auto same = [&](const char* what, const spinsum_plan_info_t& x) {
    check(x.sum_bl == before.sum_bl && x.bl == before.bl && x.variant == before.variant &&
              x.threads == before.threads && x.persistent_per_cu == before.persistent_per_cu,
          std::string(s.name) + ": " + what);
  };
  // requested tiles faster: one of them stays and is recorded
  auto own = [](const spinsum_plan_s& P) { return P.chosen; };
  g_time = [&](const spinsum_plan_s& P) { return own(P) ? 2.0f : 1.0f; };
  spinsum_tile_t best{};
  float ms = 0;
  check(spinsum_autotune(p, buf, buf, nullptr, path.c_str(), &best, &ms) == SPINSUM_OK && ms == 1.0f,
        std::string(s.name) + ": tuned to a requested tile");
  spinsum_plan_get_info(p, &after);
  check(best.bl > 0 && after.bl == best.bl && after.sum_bl == 0, std::string(s.name) + ": requested tile kept");
  // the planner's own choice faster: it stays, the plan runs as untuned, the
  // record takes the place of the other one and plans read it, and the
  // reported tile leads back to it
  g_time = [&](const spinsum_plan_s& P) { return own(P) ? 1.0f : 2.0f; };
  check(spinsum_autotune(p, buf, buf, nullptr, path.c_str(), &best, &ms) == SPINSUM_OK && ms == 1.0f,
        std::string(s.name) + ": the planner's choice was timed");
  spinsum_plan_get_info(p, &after);
  same("the planner's choice kept", after);
  check(best.bl == 0, std::string(s.name) + ": reported as the planner's choice");
  spinsum_tile_t other{before.bl, 1, 256, 0, SPINSUM_VARIANT_REG_ONESHOT, 0};
  check(spinsum_plan_set_tile(p, &other) == SPINSUM_OK, std::string(s.name) + ": set_tile");
  check(spinsum_plan_set_tile(p, &best) == SPINSUM_OK, std::string(s.name) + ": set_tile back");
  spinsum_plan_get_info(p, &after);
  same("the reported tile leads back", after);
  std::string last;
  check(lines(path, &last) == 1, std::string(s.name) + ": one record a key");
  setenv("SPINSUM_AUTOTUNE_CACHE", path.c_str(), 1);
  spinsum_plan_t q = make(s);
  spinsum_plan_get_info(q, &after);
  same("plans read the record", after);
  // with a record of a requested tile in use the planner's own choice is
  // still the candidate, not that record
  {
    std::ofstream f(path, std::ios::trunc);
    std::string key = last.substr(0, last.find(' '));
    f << key << " " << before.bl << " 1 256 0 3 0 1.0\n";
  }
  spinsum_plan_destroy(q);
  q = make(s);
  spinsum_plan_get_info(q, &after);
  check(after.variant == SPINSUM_VARIANT_REG_ONESHOT && after.sum_bl == 0, std::string(s.name) + ": recorded tile in use");
  check(spinsum_autotune(q, buf, buf, nullptr, nullptr, &best, &ms) == SPINSUM_OK && best.bl == 0 && ms == 1.0f,
        std::string(s.name) + ": the planner's choice, not the record, was timed");
  spinsum_plan_destroy(q);
  unsetenv("SPINSUM_AUTOTUNE_CACHE");
  // nothing can be timed: the plan is what it was
  for (const spinsum_tile_t& t : {best, other}) {
    check(spinsum_plan_set_tile(p, &t) == SPINSUM_OK, std::string(s.name) + ": set_tile");
    spinsum_plan_info_t was;
    spinsum_plan_get_info(p, &was);
    g_time = [](const spinsum_plan_s&) { return -1.0f; };
    check(spinsum_autotune(p, buf, buf, nullptr, nullptr, nullptr, nullptr) == SPINSUM_ERR_UNSUPPORTED,
          std::string(s.name) + ": no candidate");
    spinsum_plan_get_info(p, &after);
    check(after.sum_bl == was.sum_bl && after.bl == was.bl && after.variant == was.variant,
          std::string(s.name) + ": kept without a candidate");
  }
  spinsum_plan_destroy(p);
  std::printf("ok %s\n", s.name);
}
}  // namespace

int main(int, char** argv) {
  const std::vector<Shape> shapes = {
      {"rows_f64", {64, 33, 33, 33}, 3, SPINSUM_F64, 1},   // tile rows at any alignment
      {"rows_f32", {64, 39, 39, 39}, 3, SPINSUM_F32, 0},
      {"wide_f64", {64, 30, 30, 30}, 3, SPINSUM_F64, 1},   // wide tiles
      {"cube_f64", {512, 24, 24, 24}, 3, SPINSUM_F64, 1},  // whole cubes in place of tiles
      {"cube_oop", {512, 24, 24, 24}, 3, SPINSUM_F64, 0},  // the planner's whole cubes, persistent
  };
  for (const Shape& s : shapes) run_case(s, argv[1]);
  std::printf(g_failed ? "%d checks FAILED\n" : "PASSED\n", g_failed);
  return g_failed != 0;
}

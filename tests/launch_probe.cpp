// Lists the kernels that calls of libppf.so launch, without a GPU: this program
// defines the HIP runtime functions that the library uses, and its own
// definitions are found before the runtime's. Memory is host memory, copies
// are copies, and a launch only notes the kernel's name, its stream and the
// calling thread. Commands are lines on stdin:
//   exec|noalloc N T type path M        path 0 auto, 1 fused, 2 two-pass
//   push N T type path M
//   power N T type path M K
//   query N T type path M K             the workspace bytes after exec (K = 0) or power
//   grid exec|power N T type path M K   name:workgroups
//   threads exec|power N T type path M K stream     two threads, four calls each, on one
//                                       stream handle; every launch takes a while
// The answer is one line each: kernel names, for `threads` as thread:name;
// waits and records of events stand among the launches.

#include <hip/hip_runtime_api.h>

#include <chrono>
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

#include "ppf.h"

namespace {

std::mutex g_mu;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;      // filled before main by the library's registration
  return m;
}
std::vector<std::string> g_log;
bool g_slow = false, g_grid = false;
thread_local int t_thread = -1;

void note(const std::string& what) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_log.push_back(t_thread < 0 ? what : std::to_string(t_thread) + ":" + what);
}

// "void ppf::(anonymous namespace)::ppf_long_kernel<64, ..>(args)" -> "ppf_long_kernel<64,..>"
std::string short_name(const char* mangled) {
  int st = 0;
  char* d = abi::__cxa_demangle(mangled, nullptr, nullptr, &st);
  std::string s = st == 0 ? d : mangled;
  free(d);
  const size_t at = s.find("ppf_");
  if (at != std::string::npos) s = s.substr(at);
  std::string out;
  int depth = 0;
  for (char c : s) {
    if (c == '(' && depth == 0) break;
    if (c == '<') ++depth;
    if (c == '>') --depth;
    if (c != ' ') out += c;
  }
  return out;
}

struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
thread_local std::vector<Config> t_config;

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
  names()[host] = short_name(device);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  t_config.push_back(Config{grid, block, lds, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  const Config c = t_config.back();
  t_config.pop_back();
  *grid = c.grid; *block = c.block; *lds = c.lds; *stream = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, hipStream_t) {
  note(names()[f] + (g_grid ? ":" + std::to_string(grid.x) : ""));
  if (g_slow) std::this_thread::sleep_for(std::chrono::milliseconds(4));
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char here[256]; *p = here; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(16); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free((void*)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)malloc(16); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free((void*)e); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { note("record"); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { note("wait"); return hipSuccess; }
}

namespace {

char* const kIn = (char*)(1ull << 44);      // never read: no kernel runs
char* const kOut = (char*)(1ull << 45);

ppf_plan_t make(std::istringstream& is) {
  int n = 0, t = 0, type = 0, path = 0;
  is >> n >> t >> type >> path;
  const std::vector<float> h((size_t)n * t, 1.0f);
  ppf_plan_t p = ppf_plan_ex(n, t, h.data(), PPF_R32, 0, type, PPF_FFT_F32);
  if (p && path) ppf_plan_set_path(p, path);
  return p;
}

void call(ppf_plan_t p, const std::string& op, long long m, int k) {
  int st = PPF_OK;
  if (op == "exec") st = ppf_execute(p, kIn, kOut, m);
  else if (op == "noalloc") st = ppf_execute_noalloc(p, kIn, kOut, m);
  else if (op == "power") st = ppf_execute_power(p, kIn, (float*)kOut, m, k);
  else if (op == "push") {
    ppf_stream_t s = ppf_stream_create(p);
    const ppf_chunk c{kIn, kOut, m, 0};
    st = ppf_stream_push(s, &c);
    ppf_stream_destroy(s);
  }
  if (st != PPF_OK) note("status" + std::to_string(st));
}

}  // namespace

int main() {
  for (std::string line; std::getline(std::cin, line);) {
    std::istringstream is(line);
    std::string op, sub;
    is >> op;
    if (op == "threads" || op == "grid") is >> sub;
    ppf_plan_t p = make(is);
    g_log.clear();                              // without the plan's own launches
    long long m = 0, value = -1;
    int k = 1, stream = 0;
    is >> m >> k >> stream;
    if (!p) {
      note("no plan");
    } else if (op == "threads") {
      g_slow = true;
      std::vector<std::thread> ts;
      for (int i = 0; i < 2; ++i)
        ts.emplace_back([&, i] {
          t_thread = i;
          ppf_set_stream(p, (void*)(uintptr_t)stream);
          for (int r = 0; r < 4; ++r) call(p, sub, m, k);
        });
      for (auto& t : ts) t.join();
      g_slow = false;
    } else if (op == "grid") {
      g_grid = true;
      call(p, sub, m, k);
      g_grid = false;
    } else if (op == "query") {
      call(p, k ? "power" : "exec", m, k);
      ppf_plan_query(p, PPF_Q_WORKSPACE_BYTES, &value);
      g_log = {std::to_string(value)};
    } else {
      call(p, op, m, k);
    }
    const std::vector<std::string> got = g_log;
    if (p) ppf_destroy(p);
    for (size_t i = 0; i < got.size(); ++i) std::cout << (i ? " " : "") << got[i];
    std::cout << std::endl;
  }
}

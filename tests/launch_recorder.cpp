// Stand-ins for the HIP entry points that libtpdq.so calls, for tests without a
// GPU: every launch is recorded with the memory its kernel reads and writes
// (as its arguments give it) and none is made. Loaded with RTLD_GLOBAL before
// libtpdq.so, whose calls then come here.
#include <cxxabi.h>

#include <map>
#include <string>
#include <vector>

#include "tpdq_internal.h"

using tpdq::GemmArgs;

namespace {

// the argument of k_dense16 (gemm_actorder.hip)
struct DenseArgs {
  const uint16_t* X;
  int64_t ldx;
  int M, K, N;
  const uint16_t* W;
  const uint16_t* Wu;
  uint16_t* Y;
  int64_t ldy;
  float* part;
  int ks;
};

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::string g_log;
Config g_cfg;
constexpr uint64_t kScratchAt = (uint64_t)1 << 47;

size_t prepared(int64_t rows, int64_t K) {
  return tpdq::align_up((size_t)((rows + 15) / 16) * ((K + 127) / 128) * 4096);
}

// [rows][ld] elements of `size` bytes, `cols` of each row used
int64_t extent(int64_t rows, int64_t ld, int64_t cols, int size) { return ((rows - 1) * ld + cols) * size; }

std::string mems;
void mem(const char* kind, const void* p, int64_t bytes) {
  if (!mems.empty()) mems += ", ";
  mems += std::string("[\"") + kind + "\", " + std::to_string((uint64_t)p) + ", " + std::to_string(bytes) + "]";
}

template <typename T>
T arg(void** args, int i) { return *(T*)args[i]; }

// template arguments of a demangled kernel name
std::vector<std::string> targs(const std::string& name) {
  std::vector<std::string> v;
  const size_t a = name.find('<'), b = name.find('>');
  if (a == std::string::npos) return v;
  std::string cur;
  for (size_t i = a + 1; i < b; ++i) {
    if (name[i] == ',') {
      v.push_back(cur);
      cur.clear();
    } else if (name[i] != ' ') {
      cur += name[i];
    }
  }
  v.push_back(cur);
  return v;
}

void describe(const std::string& k, const std::vector<std::string>& t, void** args, const Config& c) {
  if (k == "k_gather_prep") {
    const int M = arg<int>(args, 2), K = arg<int>(args, 3);
    mem("r", arg<const void*>(args, 0), extent(M, arg<int64_t>(args, 1), K, 2));
    mem("w", arg<void*>(args, 6), prepared(M, K));
  } else if (k == "k_gather_plain") {
    const int M = arg<int>(args, 2), K = arg<int>(args, 3);
    mem("r", arg<const void*>(args, 0), extent(M, arg<int64_t>(args, 1), K, 2));
    mem("w", arg<void*>(args, 5), (int64_t)M * K * 2);
  } else if (k == "k_gather_rows") {
    const int M = (int)c.grid.x, K = arg<int>(args, 2);
    mem("r", arg<const void*>(args, 0), extent(M, arg<int64_t>(args, 1), K, 2));
    mem("w", arg<void*>(args, 4), (int64_t)M * K * 2);
  } else if (k == "k_ordered" || k == "k_rowmeta" || k == "k_wide" || k == "k_prefill") {
    const GemmArgs a = arg<GemmArgs>(args, 0);
    const bool decode = k == "k_ordered" || k == "k_rowmeta";
    const bool gated = !decode && k != "k_wide" && t.back() == "true";
    const bool prep = (decode && std::stoi(t[3]) == tpdq::kAGlobalPrep) || (k == "k_wide" && t[3] == "true");
    mem("r", a.X, prep ? (int64_t)prepared(a.M, a.K) : extent(a.M, a.ldx, a.K, 2));
    if (!decode && a.ks > 1)
      mem("w", a.part, (int64_t)a.ks * a.M * a.N * (gated ? 8 : 4));
    else
      mem("w", a.Y, extent(a.M, a.ldy, a.N, 2));
    if (a.Yp) mem("w", a.Yp, prepared(a.M, a.N));
  } else if (k == "k_splitk_reduce") {
    const int ks = arg<int>(args, 1), M = arg<int>(args, 2), N = arg<int>(args, 3);
    mem("r", arg<const void*>(args, 0), (int64_t)ks * M * N * (t.back() == "true" ? 8 : 4));
    mem("w", arg<void*>(args, 4), extent(M, arg<int64_t>(args, 5), N, 2));
  } else if (k == "k_dequant16") {
    const GemmArgs a = arg<GemmArgs>(args, 0);
    mem("w", arg<void*>(args, 3), (int64_t)((arg<int>(args, 2) + 15) / 16) * ((a.K + 127) / 128) * 4096);
  } else if (k == "k_dense16") {
    const DenseArgs a = arg<DenseArgs>(args, 0);
    const bool gated = t.back() == "true";
    const int64_t w = (int64_t)((a.N + 15) / 16) * ((a.K + 127) / 128) * 4096;
    mem("r", a.X, extent(a.M, a.ldx, a.K, 2));
    mem("r", a.W, w);
    if (gated) mem("r", a.Wu, w);
    if (a.ks > 1)
      mem("w", a.part, (int64_t)a.ks * a.M * a.N * (gated ? 8 : 4));
    else
      mem("w", a.Y, extent(a.M, a.ldy, a.N, 2));
  } else {
    mem("unknown", nullptr, 0);
  }
}

}  // namespace

extern "C" {

// the launches since the last call, as a JSON list
const char* recorder_take() {
  static std::string out;
  out = "[" + g_log + "]";
  g_log.clear();
  return out.c_str();
}

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  names()[host] = d ? d : name;
  free(d);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_cfg = Config{grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_cfg.grid;
  *block = g_cfg.block;
  *lds = g_cfg.lds;
  *s = g_cfg.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
  std::string full = names()[f];  // "void tpdq::(anonymous namespace)::k_x<..>(..)"
  const size_t at = full.find("::k_");
  if (at != std::string::npos) full = full.substr(at + 2);
  const size_t end = full.find('(', full.find('>') == std::string::npos ? 0 : full.find('>'));
  const std::string inst = full.substr(0, end);
  mems.clear();
  describe(inst.substr(0, inst.find('<')), targs(inst), args, Config{grid, block, lds, s});
  if (!g_log.empty()) g_log += ", ";
  g_log += "{\"kernel\": \"" + inst + "\", \"grid\": [" + std::to_string(grid.x) + ", " + std::to_string(grid.y) +
           "], \"block\": " + std::to_string(block.x) + ", \"lds\": " + std::to_string(lds) + ", \"mem\": [" + mems +
           "]}";
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)kScratchAt;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToHost) __builtin_memset(dst, 0, n);
  return hipSuccess;
}

}  // extern "C"

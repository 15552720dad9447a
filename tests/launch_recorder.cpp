// Records what the library launches, on the host: this program stands in for
// the HIP runtime, so that an entry point validates, plans and packs as always,
// and every launch is printed instead of made. Device pointers are never read.
//
// Usage: launch_recorder cap BYTES OP NX NY NZ NU NV SOD MAG PU PV OFF_V VIEWS [OP ...]
//   BYTES: memory a call may take beyond what is mapped before it (0: any); the
//   launches of such calls are not printed
//   OP: bp, fp (back- and forward projection of the whole volume), filter
//   (VIEWS views of NV rows of NU pixels)
// Prints, a line each:
//   attr KERNEL BYTES                        the LDS limit set for a kernel
//   launch KERNEL grid=X,Y block=N lds=BYTES [of forward projections: tu= tv=
//       tvp= vc= wide= mirror= rot=A,B]
//   call OP status=S trig=N                  sines and cosines taken
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>
#include <dlfcn.h>
#include <sys/resource.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../paper_1909_02724_amd/csrc/fdk_internal.h"

namespace {

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;  // filled before main
  return m;
}
long g_trig = 0, g_cap = 0;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_config;

double real_trig(const char* name, double x) {
  ++g_trig;
  using Fn = double (*)(double);
  static Fn fns[2] = {};
  Fn& f = fns[name[0] == 'c'];
  if (!f) f = reinterpret_cast<Fn>(dlsym(RTLD_NEXT, name));
  return f(x);
}

// Leaves the process `spare` bytes of address space.
void limit_memory(long spare) {
  long pages = 0;
  if (FILE* f = std::fopen("/proc/self/statm", "r")) {
    if (std::fscanf(f, "%ld", &pages) != 1) pages = 0;
    std::fclose(f);
  }
  const rlim_t most = static_cast<rlim_t>(pages) * sysconf(_SC_PAGESIZE) + spare;
  const rlimit limit{most, most};
  setrlimit(RLIMIT_AS, &limit);
}

}  // namespace

extern "C" {

double sin(double x) { return real_trig("sin", x); }
double cos(double x) { return real_trig("cos", x); }

void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*,
                           void*, void*, int*) {
  int status = 0;
  char* full = abi::__cxa_demangle(device, nullptr, nullptr, &status);
  std::string s = status == 0 ? full : device;
  std::free(full);
  // "void fdk::(anonymous namespace)::name<args>(types)" -> "name<args>"
  const std::string space = "(anonymous namespace)::";
  const size_t at = s.find(space);
  if (at != std::string::npos) s = s.substr(at + space.size());
  s = s.substr(0, s.find('('));
  for (char& c : s)
    if (c == ' ') c = '_';
  names()[host] = s;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = Config{grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *stream = g_config.stream;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value) {
  std::printf("attr %s %d\n", names()[f].c_str(), value);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return hipErrorInvalidSymbol;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
  if (g_cap) return hipSuccess;
  const std::string& name = names()[f];
  std::printf("launch %s grid=%u,%u block=%u lds=%zu", name.c_str(), grid.x, grid.y, block.x, lds);
  if (name.rfind("fp_", 0) == 0) {
    const auto& run = *static_cast<fdk::SliceRun*>(args[1]);
    const auto& fb = *static_cast<fdk::FpBatch*>(args[2]);
    const auto& ts = *static_cast<fdk::TileShape*>(args[3]);
    std::printf(" tu=%d tv=%d tvp=%d vc=%d wide=%d mirror=%d rot=%d,%d", ts.tu, ts.tv, ts.tvp, ts.vc,
                ts.wide, run.mirror, fb.rot_a, fb.rot_b);
  }
  std::printf("\n");
  return hipSuccess;
}

}  // extern "C"

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  g_cap = std::atol(argv[2]);
  for (int at = 3; at + 11 < argc; at += 12) {
    const std::string op = argv[at];
    auto i = [&](int n) { return std::atoi(argv[at + n]); };
    auto d = [&](int n) { return std::atof(argv[at + n]); };
    fdk_geometry g{};
    g.nx = i(1);
    g.ny = i(2);
    g.nz = i(3);
    g.nu = i(4);
    g.nv = i(5);
    g.sod = d(6);
    g.sdd = g.sod * d(7);
    g.du = d(8);
    g.dv = d(9);
    g.off_v = d(10);
    g.dx = g.dy = g.dz = 1.0;
    g.np = i(11);
    std::vector<double> angles(g.np);
    for (int s = 0; s < g.np; ++s) angles[s] = 0.1 + s * 6.283185307179586 / g.np;
    g.angles = angles.data();
    // Far apart, and never read.
    float* const a = reinterpret_cast<float*>(uintptr_t{1} << 40);
    float* const b = reinterpret_cast<float*>(uintptr_t{1} << 50);
    real_trig("sin", real_trig("cos", 0.0));
    if (g_cap) limit_memory(g_cap);
    g_trig = 0;
    const int st = op == "bp"   ? fdk_backproject(&g, 0, g.np, a, FDK_F32, b, 0, g.nz, FDK_SLAB_CONTIGUOUS, 1.0f, 0, nullptr)
                   : op == "fp" ? fdk_forward_project(&g, 0, g.np, a, 0, g.nz, FDK_SLAB_CONTIGUOUS, b, 1.0f, 0, nullptr)
                                : fdk_filter(&g, 0, g.np, a, b, FDK_F32, FDK_RAMLAK, nullptr);
    std::printf("call %s status=%d trig=%ld\n", op.c_str(), st, g_trig);
  }
  return 0;
}

// Stand-in for the HIP runtime calls that libvq makes, for tests of what the library launches (no GPU needed):
// this program is linked against libvq.so and its own definitions of those calls come first in the lookup, so
// nothing reaches the real runtime.  Reads one call a line from stdin,
//   op out in group_rows d k bits dtype B count cus        (op: assign, update, gemm, pack, gemv, lora: with static scratch)
// with several "out in" pairs as out1+out2+.. in1+in2+.. for gemv, and prints the status, then every launch:
//   status ; kernel gx gy gz threads a b ..  ; ..
// a, b, ..: for the kernels named below the integer arguments that the tests look at.  At the end, on stderr: how many
// times the library has taken memory from the heap.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>
#include "../../include/vq.h"

namespace {
std::map<const void*, std::string>& names() {   // filled while libvq's initialisers run
  static std::map<const void*, std::string> n;
  return n;
}
int g_cus = 256;
bool g_in_library = false;
long long g_allocations = 0;
std::ostringstream g_out;
dim3 g_grid, g_block;
size_t g_shared;
hipStream_t g_stream;

// Position and number of the trailing integer arguments of a kernel.
struct Ints { const char* kernel; int first, count; };
const Ints kInts[] = {{"gemm_tiny_kernel", 8, 3}, {"gemm_small_kernel", 8, 4}, {"gemm_kernel", 8, 6}};   // n_rb, n_cb, .., rpc, ..
}  // namespace

extern "C" {
void* __libc_malloc(size_t);
void* malloc(size_t n) {   // operator new comes here too
  g_allocations += g_in_library;
  return __libc_malloc(n);
}
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  g_grid = grid; g_block = block; g_shared = shared; g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = g_grid; *block = g_block; *shared = g_shared; *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  g_in_library = false;
  const std::string& name = names()[f];
  g_out << " ; " << name << " " << grid.x << " " << grid.y << " " << grid.z << " " << block.x * block.y * block.z;
  for (const Ints& k : kInts)
    if (name.find(k.kernel) != std::string::npos)
      for (int i = 0; i < k.count; ++i) g_out << " " << *static_cast<int32_t*>(args[k.first + i]);
  g_in_library = true;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = g_cus / 8 % 64; return hipSuccess; }   // a device per number of compute units: the library asks once per device
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(uintptr_t(1) << 40); return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
}

static std::vector<int> split(const std::string& s) {
  std::vector<int> v;
  std::istringstream in(s);
  for (std::string t; std::getline(in, t, '+');) v.push_back(std::stoi(t));
  return v;
}

int main() {
  auto ptr = [](int i) { return reinterpret_cast<void*>(uintptr_t(i + 1) << 44); };   // never read
  for (std::string line; std::getline(std::cin, line);) {
    std::istringstream in(line);
    std::string op, outs, ins;
    vq_desc d = {};
    int B, count, status = 0;
    in >> op >> outs >> ins >> d.group_rows >> d.d >> d.k >> d.index_bits >> d.codebook_dtype >> B >> count >> g_cus;
    d.group_cols = 256;
    std::vector<vq_desc> ds;
    const std::vector<int> o = split(outs), n = split(ins);
    for (size_t i = 0; i < o.size() && i < n.size(); ++i) {
      d.out_features = o[i];
      d.in_features = n[i];
      for (int c = 0; c < count; ++c) ds.push_back(d);
    }
    g_out.str("");
    g_in_library = op != "gemv" && op != "lora";
    const int ld = (B + 7) / 8 * 8;
    if (op == "assign") status = vq_em_assign(&ds[0], ptr(0), ptr(1), ptr(2), ptr(3), nullptr);
    else if (op == "update") status = vq_em_update(&ds[0], ptr(0), ptr(1), ptr(2), ptr(3), nullptr);
    else if (op == "pack") status = vq_pack_layout(&ds[0], ptr(0), ptr(1), ptr(2), ptr(3), nullptr);
    else if (op == "gemm") status = vq_gemm_batched(&ds[0], ptr(0), ptr(1), ptr(2), B, ld, ptr(3), ld, VQ_F16, nullptr);
    else if (op == "gemv" || op == "lora") {
      const std::vector<const void*> p(ds.size(), ptr(0)), x(ds.size(), ptr(1));
      const std::vector<void*> y(ds.size(), ptr(2));
      const std::vector<vq_lora_desc> adapters(ds.size(), {ptr(3), ptr(4), 16, 0});
      g_in_library = true;
      if (op == "gemv") status = vq_gemv_multi((int)ds.size(), ds.data(), p.data(), p.data(), x.data(), y.data(), VQ_F16, nullptr);
      else status = vq_gemv_lora_multi_static((int)ds.size(), ds.data(), p.data(), p.data(), x.data(), adapters.data(), y.data(), VQ_F16, nullptr);
    } else {
      std::fprintf(stderr, "unknown op %s\n", op.c_str());
      return 1;
    }
    g_in_library = false;
    std::cout << status << g_out.str() << "\n";
  }
  std::cerr << "allocations " << g_allocations << "\n";
  return 0;
}

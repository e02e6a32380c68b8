// Host-side check of the projection dispatch: launch_gemm runs over the products a
// forward can ask for, with kernel launches replaced by a recorder, and
//  - answers every one of them (no plan names a kernel that is not built),
//  - covers the output with tiles and keeps the K slices inside the scratch,
//  - takes the same tiles, K slices and order for weights as stored and as the fp16
//    image (the waves of a tile may lie differently), so that results are the same,
//  - prints the kernels it chose, one per line, for comparison with those the
//    library holds.
// With arguments "M N K epilogue part_bytes" it prints the launches of that one
// product (a residual one with the norm after it) on fp16 weights and 256 compute
// units: kernel, grid x, y, z.
#include "../../paper_2608_28099_amd/csrc/common.h"

#include <cxxabi.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <string>
#include <typeinfo>
#include <vector>

#include "../../paper_2608_28099_amd/csrc/kernels.h"

namespace {

struct Launch { std::string kernel; dim3 grid, block; };
std::vector<Launch> g_launches;

template <auto F> struct Tag {};

template <auto F>
std::string kernel_name() {  // "kernel<...>" out of "...Tag<&(sp::(anonymous namespace)::kernel<...>(...))>"
  int status = 0;
  char* d = abi::__cxa_demangle(typeid(Tag<F>).name(), nullptr, nullptr, &status);
  std::string s = status == 0 && d ? d : typeid(Tag<F>).name();
  std::free(d);
  const size_t at = s.rfind("gemm_"), end = s.find('(', at);
  return at == std::string::npos || end == std::string::npos ? s : s.substr(at, end - at);
}

// What decides the order of a launch's sums: the kernel without its wave layout and kind of weights, the grid.
std::string sums_of(const Launch& l) {
  std::vector<std::string> args;
  const size_t open = l.kernel.find('<');
  std::string s = l.kernel.substr(0, open), cur;
  for (size_t i = open + 1; open != std::string::npos && i < l.kernel.size(); ++i) {
    const char c = l.kernel[i];
    if (c == ',' || c == '>') { args.push_back(cur); cur.clear(); }
    else if (c != ' ') cur += c;
  }
  const bool lds = s == "gemm_lds", rows = s == "gemm_rows";
  for (size_t i = 0; i < args.size(); ++i) {
    if (lds && (i == 2 || i == 3)) continue;
    if ((lds || rows) && i + 1 == args.size()) continue;
    s += "," + args[i];
  }
  return s + " " + std::to_string(l.grid.x) + " " + std::to_string(l.grid.y) + ";";
}

template <auto F>
void record(dim3 grid, dim3 block) {
  static const std::string name = kernel_name<F>();
  g_launches.push_back({name, grid, block});
}

}  // namespace

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) record<kernel>(grid, block)
#define hipGetLastError() hipSuccess

#include "../../paper_2608_28099_amd/csrc/gemm.hip"

int main(int argc, char** argv) {
  using namespace sp;
  if (argc == 6) {
    char* base = reinterpret_cast<char*>((uintptr_t)0x100000000000ull);
    bool done = false;
    GemmParams p{};
    p.a = p.norm_gain = base;
    p.c = p.norm_out = base;
    p.r = p.b[0] = p.b[1] = p.b[2] = base;
    p.part = (float*)base;
    p.M = std::atoi(argv[1]); p.N = std::atoi(argv[2]); p.K = std::atoi(argv[3]);
    p.lda = p.ldb = p.K; p.ldc = p.r_ld = p.N; p.r_mod = p.M; p.norm_ld = p.N;
    p.b_split0 = p.b_split1 = p.N;
    p.b_f16 = 1; p.n_cus = 256; p.n_xcd = 8;
    p.part_bytes = std::strtoull(argv[5], nullptr, 10);
    const int epi = std::atoi(argv[4]);
    if (epi == kEpiResidRow || epi == kEpiResidF32) p.norm_done = &done;
    if (epi == kEpiSwiglu) p.ldc = p.N / 2;
    if (launch_gemm(kBF16, (Epilogue)epi, p, nullptr) != hipSuccess) return 1;
    for (const Launch& l : g_launches) std::printf("%s|%u|%u|%u\n", l.kernel.c_str(), l.grid.x, l.grid.y, l.grid.z);
    return 0;
  }
  std::set<std::string> reached;
  long products = 0, failures = 0;
  auto fail = [&](const char* what, Epilogue epi, const GemmParams& p) {
    if (failures++ < 20)
      std::fprintf(stderr, "FAIL %s: epilogue %d, %d x %d x %d, image %d, %d compute units\n", what, (int)epi, p.M, p.N,
                   p.K, p.b_f16, p.n_cus);
  };
  std::vector<int> rows, widths, depths;
  for (int m : {1, 2, 5, 8, 9, 12, 13, 16, 17, 24, 31, 32, 33, 48, 64, 65, 96, 97, 128, 129, 160, 192, 256, 257, 384, 512, 640,
                768, 1000, 1024, 1025, 1536, 2048, 3000, 4096, 8192, 16384, 40000, 65536, 100000})
    rows.push_back(m);
  for (int n = 32; n <= 1024; n += 32) widths.push_back(n);
  for (int n = 1024 + 64; n <= 8192; n += 64) widths.push_back(n);
  for (int n = 8192 + 32; n <= 40960; n += 416) widths.push_back(n);
  for (int n = 8192 + 256; n <= 40960; n += 1024) widths.push_back(n);
  for (int n : {12288, 19456, 24576, 34816, 57344, 5120 * 4, 33024, 65536}) widths.push_back(n);
  for (int k : {32, 64, 96, 128, 192, 256, 320, 512, 544, 640, 768, 1024, 1536, 2048, 2080, 2560, 3072, 4096, 4128, 4160, 5120,
                7680, 8192, 8224, 9216, 9728, 12288, 14336, 16384, 17408, 28672})
    depths.push_back(k);
  char* base = reinterpret_cast<char*>((uintptr_t)0x100000000000ull);
  for (int cus : {256, 80, 304})
    for (int e = 0; e <= (int)kEpiRowScale; ++e)
      for (int m : rows)
        for (int n : widths)
          for (int k : depths) {
            std::string sums[2];
            for (int image = 0; image < 2; ++image) {
              const Epilogue epi = (Epilogue)e;
              if (epi == kEpiSwiglu && n % 64) continue;
              if ((int64_t)m * std::max(n, k) > (int64_t)1 << 30) continue;
              GemmParams p{};
              p.a = base; p.c = base + ((size_t)1 << 40); p.r = base + ((size_t)2 << 40);
              p.b[0] = p.b[1] = p.b[2] = base + ((size_t)3 << 40);
              p.part = (float*)(base + ((size_t)4 << 40));
              p.M = m; p.N = n; p.K = k; p.lda = p.ldb = k; p.ldc = epi == kEpiSwiglu ? n / 2 : n;
              p.b_split0 = p.b_split1 = n;
              if (epi == kEpiStore && n % 384 == 0) { p.b_split0 = n / 384 * 256; p.b_split1 = n / 384 * 320; }
              p.r_mod = m; p.r_ld = n;
              p.b_f16 = image; p.n_cus = cus; p.n_xcd = 8;
              // the workspace's rule, for heads whose widest product is this one, the
              // gate/up of a down projection, or far wider
              const size_t widest[] = {(size_t)n, std::max((size_t)n, 2 * (size_t)k), (size_t)1 << 21};
              p.part_bytes = std::max((size_t)16 * 32 * widest[(m + n / 32 + k / 32) % 3], (size_t)4 * std::min(m, 1024) * n) * 4;
              p.status = (int*)base;  // (no pointer is dereferenced)
              // a residual product's norm, as the forwards ask for it
              bool done = false;
              if (epi == kEpiResidRow || epi == kEpiResidF32) {
                p.norm_gain = base + ((size_t)5 << 40); p.norm_out = base + ((size_t)6 << 40); p.norm_ld = n;
                p.norm_done = &done;
              }
              for (int norm = p.norm_done ? 1 : 0; norm >= 0; --norm) {
                if (!norm) p.norm_done = nullptr;
                g_launches.clear();
                ++products;
                if (launch_gemm(kBF16, epi, p, nullptr) != hipSuccess || g_launches.empty()) {
                  fail("refused", epi, p);
                  continue;
                }
                int64_t outputs = 0;
                for (const Launch& l : g_launches) {
                  reached.insert(l.kernel);
                  int bm, bn;
                  if (std::sscanf(l.kernel.c_str(), "gemm_lds<%d, %d", &bm, &bn) == 2) {
                    outputs += (int64_t)l.grid.x * bm * bn;
                    if (l.grid.y > 1 && (size_t)l.grid.y * m * n * 4 > p.part_bytes) fail("slices past the scratch", epi, p);
                  } else if (l.kernel.rfind("gemm_rows", 0) == 0) {
                    outputs += (int64_t)l.grid.x * l.grid.y * 16 * (epi == kEpiSwiglu ? 32 : 16);
                  }
                }
                if (outputs < (int64_t)m * n) fail("outputs left out", epi, p);
                for (const Launch& l : g_launches) sums[image] += sums_of(l);
              }
              if (image && sums[0] != sums[1]) fail("other sums with the image", epi, p);
            }
          }
  // fp32: rows past one grid dimension among them
  for (int e = 0; e <= (int)kEpiRowScale; ++e)
    for (int m : {1, 16, 17, 64, 4096, 16 * 65535, 16 * 65535 + 1, 64 * 65535 + 1})
      for (int n : {8, 72, 4096}) {
        GemmParams p{};
        p.M = m; p.N = n; p.K = p.lda = p.ldb = 36; p.n_cus = 256;
        g_launches.clear();
        ++products;
        if (launch_gemm(kF32, (Epilogue)e, p, nullptr) != hipSuccess || g_launches.size() != 1) {
          fail("fp32 refused", (Epilogue)e, p);
          continue;
        }
        const Launch& l = g_launches[0];
        int mt = 0;
        std::sscanf(l.kernel.c_str(), "gemm_f32<%d", &mt);
        reached.insert(l.kernel);
        if (l.grid.y > 65535 || l.grid.z > 65535 || (int64_t)l.grid.y * l.grid.z * 16 * mt < m) fail("fp32 grid", (Epilogue)e, p);
      }
  for (const std::string& k : reached) std::printf("%s\n", k.c_str());
  std::fprintf(stderr, "%ld products, %ld failures, %zu kernels\n", products, failures, reached.size());
  return failures ? 1 : 0;
}

// route_driver.cpp -- shows which launches the built library makes for a plan,
// on a machine without a GPU (test infrastructure).
//
// The HIP runtime's entry points of hip_stub.cpp are defined in this program,
// so libpwfs.so binds to them: device memory is host memory (the workspace is
// reserved, not committed) and kernels do not run.  Every launch is recorded;
// for the Toeplitz passes their arguments too, from which the bytes that a pass
// may touch are compared with the end of its sensor's scratch.
//
// Commands on stdin, one a line, each answered by one line:
//   plan <frames> <sensors> <hex description>...   -> rc max_chunk chunk
//   tune <mode> <chunk> <row_groups>               -> rc max_chunk chunk
//   fwd <frames>                                   -> rc launch ...
//   scratch <sensor> <delta>                       -> bytes (its recorded size, changed by delta)
//   points                                         -> points keys, as counted and as listed, per sensor
//   free                                           -> 0
// A launch is kernel:workgroups[:parts:over], parts the workgroups that share a
// pair of column blocks, over the bytes past the end of the scratch.
#define hipLaunchKernel stub_launch_kernel
#include "hip_stub.cpp"
#undef hipLaunchKernel

#include <sys/mman.h>

#include <algorithm>
#include <iostream>
#include <sstream>
#include <vector>

#include "pwfs_internal.hpp"
#include "toep_device.hpp"

namespace {
pwfs_plan_t g_plan = nullptr;
std::vector<std::string> g_seen;

// end of the scratch of the sensor whose scratch starts at p: what is recorded
// for it, at most the next sensor's or the counters
const char* scratch_end(const void* p) {
  const char* end = (const char*)g_plan->counters;
  for (const pwfs::SensorPlan& s : g_plan->s) {
    if ((const char*)s.rbuf > (const char*)p) end = std::min(end, (const char*)s.rbuf);
    if ((const char*)s.rbuf == (const char*)p) end = std::min(end, (const char*)p + s.rbuf_bytes);
  }
  return end;
}
long long over(const void* base, const void* end) {
  const long long n = (const char*)end - scratch_end(base);
  return n > 0 ? n : 0;
}
std::string short_name(const std::string& mangled) {
  for (const char* k : {"k_toep_rows_ident", "k_toep_cols_ident", "k_toep_rows", "k_toep_cols_halves", "k_toep_cols", "k_toep_sum",
                        "k_toep_field", "k_toep_hetero", "k_hetero", "k_fused", "k_rows_ident", "k_cols_ident", "k_rows",
                        "k_cols", "k_field", "k_slopes", "k_counter_reset"})
    if (mangled.find(k) != std::string::npos) return k;
  return mangled;
}
}  // namespace

extern "C" hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t shared,
                                      hipStream_t st) {
  const hipError_t e = stub_launch_kernel(fn, grid, block, args, shared, st);
  std::ostringstream s;
  const std::string name = short_name(names()[fn]);
  s << name << ':' << grid.x;
  if (e != hipSuccess) s << "!";
  if (g_plan && name == "k_toep_rows") {
    const auto& a = *(const pwfs::ToepRowArgs*)args[0];
    const size_t nf = a.lgroups / (a.Dq / 8);
    s << ":1:" << over(a.rbuf, a.rbuf + nf * a.n_lam * a.n_a * a.cblocks * pwfs::toep_block_floats(a.Dq));
  } else if (g_plan && (name == "k_toep_cols" || name == "k_toep_cols_halves")) {
    const auto& a = *(const pwfs::ToepColArgs*)args[0];
    const size_t nf = a.lgroups / a.cblocks, KS = (a.Dh + 15) / 16;
    long long o = over(a.rbuf, a.rbuf + nf * a.n_lam * a.n_a * a.cblocks * pwfs::toep_block_floats(a.Dq));
    if (a.n_parts > 1) o = std::max(o, over(a.rbuf, a.part + (size_t)a.units * a.lgroups * 2 * 8 * KS * 64));
    s << ':' << a.n_parts << ':' << o;
  }
  g_seen.push_back(s.str());
  return e;
}

int main() {
  std::string line;
  char* ws = nullptr;
  size_t bytes = 0;
  std::vector<float> io;
  auto chunk = [&](int rc) {
    pwfs_tuning t{};
    if (g_plan) pwfs_get_tuning(g_plan, &t);
    std::cout << rc << ' ' << t.max_chunk << ' ' << t.chunk << std::endl;
  };
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string cmd;
    in >> cmd;
    g_seen.clear();
    if (cmd == "plan") {
      int frames = 0, n = 0;
      in >> frames >> n;
      std::vector<pwfs_sensor_desc> d(n);
      for (auto& x : d) {
        std::string hex;
        in >> hex;
        for (size_t i = 0; i < sizeof x; ++i) ((unsigned char*)&x)[i] = (unsigned char)std::stoi(hex.substr(2 * i, 2), nullptr, 16);
      }
      int rc = pwfs_workspace_size(d.data(), n, frames, &bytes);
      if (!rc) {
        ws = (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        rc = ws == MAP_FAILED ? -99 : pwfs_plan(d.data(), n, frames, ws, bytes, nullptr, &g_plan);
      }
      chunk(rc);
    } else if (cmd == "tune") {
      pwfs_tuning t{};
      pwfs_get_tuning(g_plan, &t);
      in >> t.mode >> t.chunk >> t.row_groups;
      chunk(pwfs_set_tuning(g_plan, &t));
    } else if (cmd == "fwd") {
      int nf = 0;
      in >> nf;
      float dummy = 0.f;   // never read or written: kernels do not run
      std::cout << pwfs_forward(g_plan, &dummy, nf, &dummy, nullptr);
      for (const std::string& s : g_seen) std::cout << ' ' << s;
      std::cout << std::endl;
    } else if (cmd == "scratch") {
      int i = 0;
      long long delta = 0;
      in >> i >> delta;
      std::cout << (g_plan->s[i].rbuf_bytes += delta) << std::endl;
    } else if (cmd == "points") {
      for (const pwfs::SensorPlan& s : g_plan->s) {
        const pwfs::Geometry g = pwfs::geometry(s.desc);
        std::vector<pwfs::TiltPoint> pts;
        std::vector<double> keys;
        pwfs::tilt_points(s.desc, pts, keys);
        std::cout << g.n_mod << ' ' << g.n_a << ' ' << pts.size() << ' ' << keys.size() << ' ';
      }
      std::cout << std::endl;
    } else if (cmd == "free") {
      pwfs_destroy(g_plan);
      g_plan = nullptr;
      munmap(ws, bytes);
      std::cout << 0 << std::endl;
    }
  }
  return 0;
}

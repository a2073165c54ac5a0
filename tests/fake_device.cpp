// A device without a GPU: the HIP entry points that libfrbx uses, defined in
// this program (which the dynamic linker prefers to the runtime's), so that the
// library's own host code runs on the CPU.  Device memory is address space that
// counts against a quota, launches are written out by kernel name instead of
// being run.  Then one search through the C ABI, from key=value arguments:
//   if=f0,f1,...  J= K= B= D= dm_step= P= M= R= W=l0,l1,...  prec= recheck=
//   jit=0|1 (run-time compilation succeeds) budget=bytes quota=bytes
//   refuse=n (the n-th allocation from the search on fails)
//   mode=run|noalloc|stream|mixed chunk=APs pushes=n (mixed: a stream is begun,
//   which may fail, then the no-alloc search and a run)
// Output: "compiled <expression>" for what is compiled at run time, "prepared"
// when the search begins, from then on "kernel <name> grid <g> lds <bytes>" for
// every launch and "refused <bytes>", "mark <what>" between the steps, and
// "segments", "peak" (bytes) and "status" at the end.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <set>
#include <string>
#include <vector>

#include "../include/frbx.h"

namespace {

struct Fake {
  std::map<const void *, std::string> kernels, vars;
  std::map<const void *, void *> var_mem;
  std::map<char *, size_t> mem;
  std::set<std::string> names;
  size_t quota = size_t(1) << 40, used = 0, peak = 0;
  long n_malloc = 0, refuse = -1;   // refuse: this allocation (counted from 1) fails
  bool jit = false, log = false;
  std::map<void *, std::vector<std::string>> programs;
};
Fake &fake() {   // (first used by the library's own constructors)
  static Fake *f = new Fake;
  return *f;
}

char *space(size_t n) {
  void *p = mmap(nullptr, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (p == MAP_FAILED) abort();
  return static_cast<char *>(p);
}

struct Dim {
  unsigned x, y, z;
};

void launched(const std::string &name, unsigned grid, size_t lds) {
  if (fake().log) printf("kernel %s grid %u lds %zu\n", name.c_str(), grid, lds);
}

}  // namespace

extern "C" {

enum { kOk = 0, kNoMem = 2, kInvalid = 1 };

void **__hipRegisterFatBinary(const void *) {
  static void *m = nullptr;
  return &m;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, Dim *, Dim *,
                           int *) {
  fake().kernels[host] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *name, int, size_t size, int, int) {
  fake().vars[var] = name;
  fake().var_mem[var] = space(size);
}
static thread_local struct {
  Dim grid, block;
  size_t lds;
  void *stream;
} g_call;
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream) {
  g_call = {grid, block, lds, stream};
  return kOk;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream) {
  *grid = g_call.grid;
  *block = g_call.block;
  *lds = g_call.lds;
  *stream = g_call.stream;
  return kOk;
}
int hipLaunchKernel(const void *fn, Dim grid, Dim, void **, size_t lds, void *) {
  launched(fake().kernels[fn], grid.x, lds);
  return kOk;
}
int hipModuleLoadData(void **m, const void *) {
  *m = &fake();
  return kOk;
}
int hipModuleUnload(void *) { return kOk; }
int hipModuleGetFunction(void **fn, void *, const char *name) {
  *fn = const_cast<char *>(fake().names.insert(name).first->c_str());
  return kOk;
}
int hipModuleLaunchKernel(void *fn, unsigned gx, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned lds, void *,
                          void **, void **) {
  launched(std::string("jit:") + static_cast<const char *>(fn), gx, lds);
  return kOk;
}
int hipMalloc(void **p, size_t n) {
  Fake &f = fake();
  ++f.n_malloc;
  if (f.n_malloc == f.refuse || f.used + n > f.quota) {
    if (f.log) printf("refused %zu\n", n);
    *p = nullptr;
    return kNoMem;
  }
  char *m = space(n);
  f.mem[m] = n;
  f.used += n;
  if (f.used > f.peak) f.peak = f.used;
  *p = m;
  return kOk;
}
int hipFree(void *p) {
  Fake &f = fake();
  const auto it = f.mem.find(static_cast<char *>(p));
  if (!p) return kOk;
  if (it == f.mem.end()) {
    printf("free of an address that is not allocated\n");
    exit(3);
  }
  f.used -= it->second;
  munmap(p, it->second + 4096);
  f.mem.erase(it);
  return kOk;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
  memcpy(d, s, n);
  return kOk;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
  memcpy(d, s, n);
  return kOk;
}
int hipMemset(void *, int, size_t) { return kOk; }   // (fresh memory is zero)
int hipMemsetAsync(void *d, int v, size_t n, void *) {
  memset(d, v, n);
  return kOk;
}
int hipSetDevice(int) { return kOk; }
int hipGetDevice(int *d) {
  *d = 0;
  return kOk;
}
int hipGetDeviceCount(int *n) {
  *n = 1;
  return kOk;
}
int hipGetLastError(void) { return kOk; }
const char *hipGetErrorString(int) { return "fake device"; }
int hipStreamSynchronize(void *) { return kOk; }
int hipEventCreate(void **e) {
  *e = &fake();
  return kOk;
}
int hipEventDestroy(void *) { return kOk; }
int hipEventRecord(void *, void *) { return kOk; }
int hipEventElapsedTime(float *ms, void *, void *) {
  *ms = 0.f;
  return kOk;
}
int hipPointerGetAttributes(void *, const void *) { return kInvalid; }
int hipDeviceGetAttribute(int *v, int, int) {
  *v = 256;
  return kOk;
}
int hipFuncSetAttribute(const void *, int, int) { return kOk; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 1;
  return kOk;
}
int hipGetSymbolAddress(void **p, const void *var) {
  *p = fake().var_mem[var];
  return *p ? kOk : kInvalid;
}

int hiprtcCreateProgram(void **prog, const char *, const char *, int, const char **, const char **) {
  *prog = new int(0);
  return kOk;
}
int hiprtcDestroyProgram(void **) { return kOk; }
int hiprtcAddNameExpression(void *prog, const char *expr) {
  fake().programs[prog].push_back(expr);
  return kOk;
}
int hiprtcCompileProgram(void *prog, int, const char **) {
  for (const std::string &e : fake().programs[prog]) printf("compiled %s\n", e.c_str());
  return fake().jit ? 0 : 6;
}
int hiprtcGetLoweredName(void *, const char *expr, const char **name) {
  *name = fake().names.insert(expr).first->c_str();
  return kOk;
}
int hiprtcGetCodeSize(void *, size_t *n) {
  *n = 16;
  return kOk;
}
int hiprtcGetCode(void *, char *) { return kOk; }
int hiprtcGetProgramLogSize(void *, size_t *n) {
  *n = 0;
  return kOk;
}
int hiprtcGetProgramLog(void *, char *) { return kOk; }
const char *hiprtcGetErrorString(int) { return "fake compiler"; }

}  // extern "C"

int main(int argc, char **argv) {
  std::map<std::string, std::string> arg = {
      {"J", "32"},     {"K", "200"},    {"B", "1"},   {"D", "1"},      {"dm_step", "0"}, {"P", "4"},
      {"M", "256"},    {"R", "1"},      {"W", "2,4"}, {"prec", "0"},   {"recheck", "0"}, {"jit", "1"},
      {"budget", "0"}, {"quota", "0"},  {"refuse", "0"}, {"mode", "run"}, {"chunk", "64"}, {"pushes", "3"}};
  for (int i = 1; i < argc; ++i) {
    const char *eq = strchr(argv[i], '=');
    if (!eq) return 2;
    arg[std::string(argv[i], size_t(eq - argv[i]))] = eq + 1;
  }
  auto num = [&](const char *k) { return atoll(arg[k].c_str()); };
  auto list = [&](const char *k) {
    std::vector<double> v;
    for (char *p = const_cast<char *>(arg[k].c_str()); *p;) {
      v.push_back(strtod(p, &p));
      if (*p == ',') ++p;
    }
    return v;
  };
  Fake &f = fake();
  f.jit = num("jit") != 0;
  const std::vector<double> f0 = list("if");
  std::vector<int32_t> win;
  for (double w : list("W")) win.push_back(int32_t(w));
  frbx_layout lay;
  memset(&lay, 0, sizeof lay);
  lay.n_baselines = int32_t(num("B"));
  lay.n_if = int32_t(f0.size());
  lay.n_chan = int32_t(num("J"));
  lay.n_frames = num("K");
  lay.t_ap_ms = 1.0;
  lay.chan_bw_mhz = 32.0 / double(lay.n_chan);
  lay.if_freq_mhz = f0.data();
  frbx_ctx *c = nullptr;
  frbx_status s = frbx_create(&lay, 0, nullptr, &c);
  auto check = [&](const char *what) {
    if (s == FRBX_OK) return;
    printf("status %d %s: %s\n", int(s), what, frbx_last_error(c));
    exit(0);
  };
  check("create");
  s = frbx_set_dm_grid(c, 0.0, atof(arg["dm_step"].c_str()), int32_t(num("D")), 4.149e6), check("dm grid");
  s = frbx_set_delay_grid(c, int32_t(num("P")), int32_t(num("M")), 0.0, NAN), check("delay grid");
  s = frbx_set_rate_grid(c, int32_t(num("R")), 0.0), check("rate grid");
  s = frbx_set_windows(c, win.data(), int32_t(win.size())), check("windows");
  s = frbx_set_precision(c, int32_t(num("prec"))), check("precision");
  s = frbx_set_recheck(c, atof(arg["recheck"].c_str())), check("recheck");
  if (num("budget")) s = frbx_set_tile_budget(c, num("budget")), check("budget");
  const size_t n = size_t(lay.n_baselines) * f0.size() * size_t(lay.n_chan) * 8;
  const bool stream = arg["mode"] == "stream";
  int64_t len = 0;
  if (stream) {
    s = frbx_stream_begin(c, num("chunk")), check("stream begin");
  } else {
    s = frbx_load(c, space(n * size_t(lay.n_frames)), 0), check("load");
    s = frbx_get_segments(c, nullptr, nullptr, nullptr, &len), check("segments");
  }
  printf("prepared %ld\n", f.n_malloc);
  f.log = true;
  const size_t before = f.used;
  f.peak = f.used;
  if (num("quota")) f.quota = before + size_t(num("quota"));
  if (num("refuse")) f.refuse = f.n_malloc + num("refuse");
  const bool mixed = arg["mode"] == "mixed";
  if (mixed) printf("mark stream %d\n", int(frbx_stream_begin(c, num("chunk"))));
  if (mixed || arg["mode"] == "noalloc") {
    const int64_t cap = len * lay.n_baselines * num("D");
    int64_t got = 0;
    s = frbx_run_cube_noalloc(c, reinterpret_cast<float *>(space(size_t(cap) * 4)),
                              reinterpret_cast<int32_t *>(space(size_t(cap) * 4)), cap, &got);
    check("noalloc");
    if (mixed) {
      printf("mark run\n");
      s = frbx_run(c), check("run");
    }
  } else if (stream) {
    const char *chunk = space(n * size_t(num("chunk")));
    for (int i = 0; i < num("pushes"); ++i) {
      printf("mark push %d\n", i);
      s = frbx_stream_push(c, chunk, FRBX_IN_C64, nullptr, 0), check("push");
    }
  } else {
    s = frbx_run(c), check("run");
    printf("mark again\n");
    s = frbx_run(c), check("run again");
  }
  printf("segments %lld\npeak %zu\nstatus 0\n", static_cast<long long>(len), f.peak - before);
  frbx_destroy(c);
  return f.mem.empty() ? 0 : 4;
}

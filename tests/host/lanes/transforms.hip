// Runs the spectral part of plans on the matrix-core transforms without a
// GPU: the engine's own host code (plan, tables, work lists, launches) over
// host memory, the kernels from lanes.cpp.  Every buffer of a kernel (fields,
// spectral planes, tables, descriptors' control block) ends at a page that
// cannot be touched and starts after one, so that an index out of range stops
// the process.
//
// Input, one case after the other: "n0 n1 n2 prec scheme green bc[18] terms
// seed"; terms: entries of the Anderson combination (alpha) and of the
// increments taken off (beta).  Output per case, binary, into the file
// given: the combined input x and the operator's result, 3 Nn doubles each; on
// stdout a line per case (and "refused" after one whose plan is refused).
#include "../../../paper_2607_05929_amd/csrc/fm_engine.hip"

#include <csignal>
#include <cstdio>
#include <random>
#include <sys/mman.h>

// device calls of the engine that a plan and its launches make
extern "C" {
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { std::printf("FAULT other kernel launched\n"); std::fflush(stdout); std::_Exit(4); }
}

namespace {

constexpr size_t PAGE = 4096;
struct Map { char* m; size_t len, step, slack; };
std::vector<Map> maps;

// n slots of `bytes` bytes, each between two pages without access (the bytes
// from the first one to the slot are looked at afterwards), filled with NaN;
// step: the distance of two slots
char* guarded(size_t bytes, int n, size_t& step) {
  const size_t body = (bytes + PAGE - 1) / PAGE * PAGE;
  step = body + PAGE;
  const size_t len = PAGE + n * step;
  char* m = (char*)mmap(nullptr, len, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == MAP_FAILED) std::abort();
  std::memset(m, 0xff, len);
  for (int i = 0; i <= n; ++i) mprotect(m + i * step, PAGE, PROT_NONE);
  maps.push_back({m, len, step, body - bytes});
  return m + PAGE + body - bytes;
}

[[noreturn]] void stop(int code) {
  std::fflush(stdout);
  std::_Exit(code);
}

void on_fault(int) {
  static const char msg[] = "FAULT access out of range\n";
  (void)!write(1, msg, sizeof(msg) - 1);
  std::_Exit(2);
}

template <typename R>
int run(fm_plan* p, int terms, unsigned seed, std::vector<double>& x, std::vector<double>& out) {
  const Geometry& g = p->g;
  Group& G = *p->self;
  Ctrl* c = (Ctrl*)(p->ws + p->lay.ctrl);
  std::mt19937_64 rng(seed);
  std::normal_distribution<double> nd;
  std::memset(c, 0, sizeof(Ctrl));
  c->status = ST_RUNNING;
  c->depth = p->d.aa_depth;
  c->n_d = terms; c->n_b = terms - 1;
  c->slot_w = terms - 1;
  for (int i = 0; i < terms; ++i) { c->slot_d[i] = i; c->alpha[i] = terms == 1 ? 1.0 : 0.75 - 0.5 * i; }
  for (int i = 0; i + 1 < terms; ++i) { c->slot_b[i] = i; c->beta[i] = 0.25 + 0.5 * i; }
  size_t step;
  Ctrl* cg = (Ctrl*)guarded(sizeof(Ctrl), 1, step);
  *cg = *c;
  x.assign(3 * g.Nn, 0.0);
  out.assign(3 * g.Nn, 0.0);
  std::vector<char*> T(3);
  std::vector<R*> delta(3);
  std::vector<double*> uf(3);
  std::vector<size_t> dstep(3);
  for (int q = 0; q < 3; ++q) {
    T[q] = guarded(sizeof(R) * g.s1[q], 1, step);
    const size_t fb = sizeof(R) * g.Nn;
    char* ring = guarded(fb, terms, step);
    delta[q] = (R*)guarded(fb, terms, dstep[q]);
    uf[q] = (double*)guarded(8 * g.Nn, 1, dstep[q]);
    dstep[q] = step;
    for (int64_t i = 0; i < g.Nn; ++i) {
      const int J[3] = {(int)(i % g.N[0]), (int)(i / g.N[0] % g.N[1]), (int)(i / g.N[0] / g.N[1])};
      bool kept = true;
      for (int a = 0; a < 3; ++a) {
        int j0, cnt;
        raw_range(g.kinds[q][a], g.n[a], j0, cnt);
        kept = kept && J[a] >= j0 && J[a] < j0 + cnt;
      }
      uf[q][i] = 0;
      // (what dismissed nodes hold must not enter)
      for (int t = 0; t < terms; ++t) {
        R* r = (R*)(ring + t * step) + i;
        *r = (R)(kept ? nd(rng) : 1e3 * nd(rng));
        if (kept) x[q * g.Nn + i] += (double)(R)cg->alpha[t] * *r;
        if (t + 1 < terms) ((R*)((char*)delta[q] + t * step))[i] = kept ? (R)nd(rng) : (R)0;
      }
    }
    std::map<const void*, char*> tab;
    MatDesc& d = G.M[q];
    d.ctrl = cg;
    d.D = ring;
    d.delta = delta[q];
    d.ring_stride = step / sizeof(R);
    d.T = T[q];
    d.uf = uf[q];
    for (MatAxis& m : d.x) {
      auto move = [&](const void*& t, size_t bytes) {
        char*& to = tab[t];
        size_t s;
        if (!to) { to = guarded(bytes, 1, s); std::memcpy(to, t, bytes); }
        t = to;
      };
      const size_t half = (size_t)m.kt * m.kt * 256 * sizeof(R);
      move(m.fU, half); move(m.fV, half); move(m.iU, half); move(m.iV, half);
      const void* gs = m.gs;
      move(gs, (size_t)64 * m.kt * 8);
      m.gs = (const double*)gs;
      move(m.gz, (size_t)64 * m.kt * sizeof(R));
    }
  }
  for (int slot : {0, 1, 2, 3, 4})
    if (int rc = launch_slot<R>(G, slot)) return rc;
  for (int q = 0; q < 3; ++q)
    for (int64_t i = 0; i < g.Nn; ++i) {
      // the increment, in the ring and added once to the displacement
      const R w = ((R*)((char*)delta[q] + (terms - 1) * dstep[q]))[i];
      if (!(uf[q][i] == (double)w)) { std::printf("FAULT node %d %lld: displacement %g increment %g\n", q, (long long)i, uf[q][i], (double)w); stop(5); }
      double v = w;
      for (int t = 0; t + 1 < terms; ++t) v += (double)(R)cg->beta[t] * ((R*)((char*)delta[q] + t * dstep[q]))[i];
      out[q * g.Nn + i] = v;
    }
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  std::signal(SIGSEGV, on_fault);
  FILE* f = argc > 1 ? std::fopen(argv[1], "wb") : nullptr;
  fm_plan_desc d;
  std::memset(&d, 0, sizeof(d));
  d.h = 1.0; d.lambda0 = 1.25; d.mu0 = 0.75; d.tol = 1e-6;
  d.max_iter = 10; d.aa_depth = 4; d.aa_period = 3; d.max_materials = 2;
  int v[6], terms, seed;
  while (std::scanf("%d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5) == 6) {
    for (int i = 0; i < 3; ++i) d.n[i] = v[i];
    d.prec = v[3]; d.scheme = v[4]; d.green = v[5];
    int* bc = &d.bc[0][0][0];
    for (int i = 0; i < 18; ++i)
      if (std::scanf("%d", bc + i) != 1) return 1;
    if (std::scanf("%d %d", &terms, &seed) != 2) return 1;
    std::printf("case %d x %d x %d prec %d scheme %d terms %d\n", v[0], v[1], v[2], v[3], v[4], terms);
    std::fflush(stdout);
    const size_t bytes = fm_workspace_bytes(&d);
    std::vector<char> ws(bytes + 4096, (char)0xff);
    fm_plan* p = nullptr;
    if (!bytes && std::strstr(fm_last_error(), "too long")) {      // a pencil the plan does not take
      std::printf("refused\n");
      continue;
    }
    if (!bytes || fm_plan_create(&d, (char*)(((uintptr_t)ws.data() + 255) / 256 * 256), bytes, nullptr, &p)) {
      std::printf("FAULT %s\n", fm_last_error());
      return 6;
    }
    if (!p->g.mat) { std::printf("FAULT not on the matrix cores\n"); return 7; }
    std::vector<double> x, out;
    if (d.prec == FM_FP64 ? run<double>(p, terms, seed, x, out) : run<float>(p, terms, seed, x, out)) {
      std::printf("FAULT %s\n", fm_last_error());
      return 8;
    }
    if (f) { std::fwrite(x.data(), 8, x.size(), f); std::fwrite(out.data(), 8, out.size(), f); }
    fm_plan_destroy(p);
    for (auto& m : maps) {
      for (size_t at = PAGE; at < m.len; at += m.step)
        for (size_t i = 0; i < m.slack; ++i)
          if (m.m[at + i] != (char)0xff) { std::printf("FAULT write before a buffer\n"); stop(9); }
      munmap(m.m, m.len);
    }
    maps.clear();
  }
  if (f) std::fclose(f);
  std::printf("done\n");
  return 0;
}

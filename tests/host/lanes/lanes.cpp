// The matrix-core transforms on the host, and the scheduler of their lanes.
#include "../../../paper_2607_05929_amd/csrc/fm_mat.hip"

#include <sys/mman.h>

#include <vector>

namespace fm {
namespace {
__attribute__((aligned(4096))) char smem[192 * 1024];     // the kernels' dynamic LDS
}
}  // namespace fm

extern "C" void lanes_switch(void** from, void* to);
asm(R"(
.text
.globl lanes_switch
lanes_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

namespace lanes {
namespace {
constexpr size_t STACK = 128 * 1024;
std::vector<Lane> lane;
char* stacks = nullptr;
void* scheduler;
size_t cur;
const std::function<void()>* job;

void start() {
  (*job)();
  yield(W_DONE);
  stop("resumed after its end");
}

// every lane of a wavefront or block waits for the same
Wait common(size_t first, size_t n) {
  for (size_t i = 1; i < n; ++i)
    if (lane[first + i].wait != lane[first].wait) {
      thread_idx.x = (unsigned)(first + i);
      stop("divergent wait");
    }
  return lane[first].wait;
}

template <typename R>
void product(Lane* w) {
  R d[16][16];
  for (int i = 0; i < 16; ++i)
    for (int j = 0; j < 16; ++j) {
      const int g = sizeof(R) == 4 ? i >> 2 : i & 3, r = sizeof(R) == 4 ? i & 3 : i >> 2;
      R s = (R)w[16 * g + j].c[r];
      for (int k = 0; k < 4; ++k) {
        const double a = w[16 * k + i].a, b = w[16 * k + j].b;
        s = sizeof(R) == 4 ? (R)(a * b + (double)s) : (R)std::fma(a, b, (double)s);
      }
      d[i][j] = s;
    }
  for (int l = 0; l < 64; ++l)
    for (int r = 0; r < 4; ++r) w[l].c[r] = d[sizeof(R) == 4 ? 4 * (l >> 4) + r : 4 * r + (l >> 4)][l & 15];
}
}  // namespace

Lane& self() { return lane[cur]; }

void yield(Wait w) {
  lane[cur].wait = w;
  lanes_switch(&lane[cur].sp, scheduler);
}

void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()>& body) {
  const size_t n = block.x;
  if (n % 64 || n > 1024 || lds > 160 * 1024) stop("launch shape");
  if (!stacks)
    stacks = (char*)mmap(nullptr, 1024 * STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  lane.resize(n);
  job = &body;
  block_dim = {block.x, 1, 1};
  for (unsigned b = 0; b < grid.x; ++b) {
    block_idx = {b, 0, 0};
    std::memset(fm::smem, 0xff, sizeof(fm::smem));
    for (size_t i = 0; i < n; ++i) {
      void** sp = (void**)(stacks + (i + 1) * STACK);
      *--sp = nullptr;                       // (keeps the entry's stack alignment)
      *--sp = (void*)start;
      for (int r = 0; r < 6; ++r) *--sp = nullptr;
      lane[i].sp = sp;
      lane[i].wait = W_RUN;
    }
    size_t done = 0;
    while (done < n) {
      // one wavefront after the other to its next barrier or its end
      for (size_t w = 0; w < n; w += 64) {
        if (lane[w].wait == W_DONE) continue;
        do {
          for (cur = w; cur < w + 64; ++cur) {
            thread_idx = {(unsigned)cur, 0, 0};
            lanes_switch(&scheduler, lane[cur].sp);
          }
          if (common(w, 64) == W_MFMA) {
            if (lane[w].prec == 4) product<float>(&lane[w]);
            else product<double>(&lane[w]);
          }
        } while (lane[w].wait == W_MFMA);
        if (lane[w].wait == W_DONE) done += 64;
      }
      if (done && done < n) {
        // (whole wavefronts may end early, but then none may reach a barrier)
        for (size_t w = 0; w < n; w += 64)
          if (lane[w].wait == W_BARRIER) stop("barrier not reached by every wavefront");
      }
    }
    for (size_t i = lds; i < sizeof(fm::smem); ++i)
      if (fm::smem[i] != (char)0xff) stop("write past the dynamic LDS");
  }
}

}  // namespace lanes

// Blocks of a kernel on the host: each lane is a coroutine; a matrix
// instruction collects the operands of its 64 lanes, a barrier every lane of
// the block.  The dynamic LDS starts as NaN and ends in bytes that must stay
// as they are.
#pragma once
#include <cstdio>
#include <cstdlib>
#include <functional>

namespace lanes {

struct Idx { unsigned x, y, z; };
inline Idx thread_idx, block_idx, block_dim;

enum Wait : int { W_RUN, W_MFMA, W_BARRIER, W_DONE };
struct Lane {
  void* sp;
  Wait wait;
  unsigned prec;          // reals of the matrix instruction: 4 or 8 bytes
  double a, b, c[4];
};

[[noreturn]] inline void stop(const char* what) {
  std::printf("FAULT %s: block %u thread %u\n", what, block_idx.x, thread_idx.x);
  std::fflush(stdout);
  std::_Exit(3);
}

void yield(Wait w);
Lane& self();
void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()>& body);
inline void barrier() { yield(W_BARRIER); }

// D = A B + C of 16 x 16 x 4: lane l holds A[l & 15][l >> 4], B[l >> 4][l & 15] and
// column l & 15 of C and D (rows 4 (l >> 4) + r in FP32, 4 r + (l >> 4) in FP64)
template <typename R, typename V>
V mfma(R a, R b, V c) {
  Lane& l = self();
  l.prec = sizeof(R);
  l.a = a; l.b = b;
  for (int r = 0; r < 4; ++r) l.c[r] = c[r];
  yield(W_MFMA);
  for (int r = 0; r < 4; ++r) c[r] = (R)l.c[r];
  return c;
}

}  // namespace lanes

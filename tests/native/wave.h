// A wave of 64 lanes on the CPU: every lane is a fiber that runs to the next
// cross-lane operation, leaves its value there and lets the next lane run, so
// that all values of an operation are there before the first lane goes on.
// Lanes that meet at different operations end the process: the code was not
// wave-uniform where it has to be.
#pragma once

#include <setjmp.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#include "hip/hip_runtime.h"

namespace wave {

constexpr int LANES = 64;
constexpr size_t STACK = 1 << 16;

struct Fiber {
  jmp_buf at;  // where the lane goes on: at an operation, or at the next run
  std::vector<char> stack;
};
inline Fiber fibers[LANES];
inline jmp_buf main_at;
inline int cur, ended;
inline uint64_t count[LANES];  // operations of each lane
inline uint32_t value[2][LANES];
inline int code[2][LANES];
inline std::function<void(int)> body;

inline void next() {
  cur = (cur + 1) % LANES;
  _longjmp(fibers[cur].at, 1);
}

inline void entry() {
  volatile const int lane = cur;
  volatile bool made = false;
  for (;;) {
    // wait for a run; the lane that ends the last gives control back
    if (_setjmp(fibers[lane].at) == 0) {
      if (!made || ++ended == LANES) _longjmp(main_at, 1);
      next();
    }
    made = true;
    body(lane);
    if (count[lane] != count[0]) {
      fprintf(stderr, "lane %d ended after %llu operations, lane 0 after %llu\n", lane, (unsigned long long)count[lane],
              (unsigned long long)count[0]);
      abort();
    }
  }
}

// Leave v at the operation; returns all lanes' values once they are there.
inline const uint32_t* exchange(int op, uint32_t v) {
  const int lane = cur, k = (int)(count[lane]++ & 1);
  value[k][lane] = v;
  code[k][lane] = op;
  if (_setjmp(fibers[lane].at) == 0) next();
  for (int i = 0; i < LANES; ++i)
    if (code[k][i] != op) {
      fprintf(stderr, "lanes %d and %d meet at different operations (%d, %d)\n", lane, i, op, code[k][i]);
      abort();
    }
  return value[k];
}

// Run f(lane) on every lane of one wave.
template <class F>
void run(F f) {
  body = f;
  if (fibers[0].stack.empty())
    for (cur = 0; cur < LANES; ++cur) {
      fibers[cur].stack.resize(STACK);
      ucontext_t c;
      getcontext(&c);
      c.uc_stack.ss_sp = fibers[cur].stack.data();
      c.uc_stack.ss_size = STACK;
      c.uc_link = nullptr;
      makecontext(&c, entry, 0);
      if (_setjmp(main_at) == 0) setcontext(&c);
    }
  cur = ended = 0;
  for (int i = 0; i < LANES; ++i) count[i] = 0;
  if (_setjmp(main_at) == 0) _longjmp(fibers[0].at, 1);
}

}  // namespace wave

inline LaneIndex::operator uint32_t() const { return (uint32_t)wave::cur; }
inline ThreadIndex threadIdx;

inline uint64_t __ballot(bool x) {
  const uint32_t* v = wave::exchange(1, x);
  uint64_t m = 0;
  for (int i = 0; i < wave::LANES; ++i) m |= (uint64_t)(v[i] != 0u) << i;
  return m;
}
inline int __builtin_amdgcn_readlane(int x, int lane) { return (int)wave::exchange(2, (uint32_t)x)[lane & 63]; }
inline int __builtin_amdgcn_readfirstlane(int x) { return (int)wave::exchange(3, (uint32_t)x)[0]; }
inline int __builtin_amdgcn_update_dpp(int old, int src, int ctrl, int row_mask, int bank_mask, bool bound_ctrl) {
  const uint32_t* v = wave::exchange(0x10000 + ctrl, (uint32_t)src);
  const int lane = wave::cur, row = lane & ~15, in = lane & 15;
  int from = -1;
  if (ctrl < 0x100) from = (lane & ~3) | ((ctrl >> (2 * (lane & 3))) & 3);      // quad_perm
  else if (ctrl > 0x110 && ctrl < 0x120) from = in >= (ctrl & 15) ? lane - (ctrl & 15) : -1;  // row_shr
  else if (ctrl == 0x130) from = lane < 63 ? lane + 1 : -1;                      // wave_shl:1
  else if (ctrl == 0x138) from = lane - 1;                                       // wave_shr:1
  else if (ctrl == 0x140) from = row + 15 - in;                                  // row_mirror
  else if (ctrl == 0x141) from = (lane & ~7) + 7 - (lane & 7);                   // row_half_mirror
  else if (ctrl == 0x142) from = row - 1;                                        // row_bcast:15
  else if (ctrl == 0x143) from = lane >= 32 ? 31 : -1;                           // row_bcast:31
  else abort();
  if (!((row_mask >> (lane >> 4)) & 1) || !((bank_mask >> (in >> 2)) & 1)) return old;
  if (from < 0) return bound_ctrl ? 0 : old;
  return (int)v[from];
}
inline int __builtin_amdgcn_ds_bpermute(int addr, int x) { return (int)wave::exchange(4, (uint32_t)x)[(addr >> 2) & 63]; }
inline u32pair __builtin_amdgcn_permlane16_swap(uint32_t a, uint32_t, bool, bool) {  // (both operands the same)
  const uint32_t* v = wave::exchange(5, a);
  const int i = wave::cur & 15, r = wave::cur & 32;
  return u32pair{v[r + i], v[r + 16 + i]};
}
inline u32pair __builtin_amdgcn_permlane32_swap(uint32_t a, uint32_t, bool, bool) {
  const uint32_t* v = wave::exchange(6, a);
  return u32pair{v[wave::cur & 31], v[32 + (wave::cur & 31)]};
}
inline bool __builtin_amdgcn_inverse_ballot_w64(uint64_t m) { return (m >> wave::cur) & 1u; }
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t add) {
  return add + (uint32_t)__builtin_popcount(wave::cur >= 32 ? m : m & ((1u << wave::cur) - 1u));
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t add) {
  return add + (wave::cur > 32 ? (uint32_t)__builtin_popcount(m & ((1u << (wave::cur - 32)) - 1u)) : 0u);
}
inline int __shfl_down(int x, int d, int) {
  const uint32_t* v = wave::exchange(7, (uint32_t)x);
  return (int)v[wave::cur + d < 64 ? wave::cur + d : wave::cur];
}
inline void __syncthreads() { abort(); }  // (one wave)

// Workgroups on the host CPU: one fiber per thread. A fiber runs until its lane has to wait for others -- a value from
// another lane, a barrier -- and when nobody can go on, the waves and then the barrier that are complete let go. What
// waits for lanes that never come ends the process.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <vector>

namespace emu {
dim3 thread_idx, block_idx, block_dim, grid_dim;

namespace {
constexpr size_t kStack = 256 << 10;
enum State { kRuns, kWaitsWave, kWaitsBlock, kDone };
struct Fiber {
  ucontext_t at;
  State state;
  int parity;
};
struct Wave {
  alignas(64) char slot[2][64][64];
};
std::vector<Fiber> fibers;
std::vector<Wave> waves;
char *stacks = nullptr;
ucontext_t scheduler;
int current = -1;
const std::function<void()> *work = nullptr;
void (*hook)(int block, int barrier) = nullptr;

void fiber_main() {
  (*work)();
  fibers[current].state = kDone;
  swapcontext(&fibers[current].at, &scheduler);
}
void wait(State s) {
  fibers[current].state = s;
  const int me = current;
  swapcontext(&fibers[me].at, &scheduler);
}

void run_block(int n) {
  for (int i = 0; i < n; ++i) {
    Fiber &f = fibers[i];
    getcontext(&f.at);
    f.at.uc_stack.ss_sp = stacks + kStack * i;
    f.at.uc_stack.ss_size = kStack;
    f.at.uc_link = nullptr;
    makecontext(&f.at, fiber_main, 0);
    f.state = kRuns;
    f.parity = 0;
  }
  for (int barriers = 0;;) {
    int done = 0, at_barrier = 0;
    for (int i = 0; i < n; ++i) {
      if (fibers[i].state != kRuns) continue;
      current = i;
      thread_idx.x = i;
      swapcontext(&scheduler, &fibers[i].at);
    }
    bool moved = false;
    for (int w = 0; w * 64 < n; ++w) {
      int here = 0, live_lanes = 0;
      for (int i = 64 * w; i < n && i < 64 * (w + 1); ++i) {
        live_lanes += fibers[i].state != kDone;
        here += fibers[i].state == kWaitsWave;
        at_barrier += fibers[i].state == kWaitsBlock;
        done += fibers[i].state == kDone;
      }
      if (here == 0 || here != live_lanes) continue;
      for (int i = 64 * w; i < n && i < 64 * (w + 1); ++i)
        if (fibers[i].state == kWaitsWave) fibers[i].state = kRuns;
      moved = true;
    }
    if (moved) continue;
    if (done == n) return;
    if (at_barrier != n - done) {
      fprintf(stderr, "lanes wait for lanes that do not come\n");
      abort();
    }
    if (hook) hook((int)(block_idx.x + block_idx.y * grid_dim.x), barriers);
    ++barriers;
    for (int i = 0; i < n; ++i)
      if (fibers[i].state == kWaitsBlock) fibers[i].state = kRuns;
  }
}
}  // namespace

int lane() { return current & 63; }
uint64_t live() {
  uint64_t m = 0;
  for (int i = current & ~63; i < (int)fibers.size() && i < (current & ~63) + 64; ++i)
    if (fibers[i].state != kDone) m |= 1ull << (i & 63);
  return m;
}
void barrier() { wait(kWaitsBlock); }
const void *exchange(const void *value, size_t bytes) {
  Wave &w = waves[current / 64];
  Fiber &f = fibers[current];
  const int slot = f.parity;
  f.parity ^= 1;
  memcpy(w.slot[slot][lane()], value, bytes);
  wait(kWaitsWave);
  return w.slot[slot];
}

Pair swap_halves(uint32_t x, uint32_t y, int width) {
  const uint32_t both[2] = {x, y};
  const char *all = static_cast<const char *>(exchange(both, sizeof both));
  const auto at = [&](int l, int which) {
    uint32_t v;
    memcpy(&v, all + 64 * l + 4 * which, sizeof v);
    return v;
  };
  const int l = lane();
  const bool odd = l & width;  // odd rows of the first operand change places with the even rows of the second
  return odd ? Pair{{at(l ^ width, 1), y}} : Pair{{x, at(l ^ width, 0)}};
}

int update_dpp(int old, int src, int ctrl, int row_mask) {
  const char *all = static_cast<const char *>(exchange(&src, sizeof src));
  const int l = lane(), row = l / 16, in_row = l % 16;
  int at = -1;
  if (ctrl < 0x100) at = (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3);
  else if (ctrl > 0x110 && ctrl < 0x120) at = in_row >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
  else if (ctrl == 0x140) at = 16 * row + 15 - in_row;
  else if (ctrl == 0x141) at = (l & ~7) | (7 - (l & 7));
  else if (ctrl == 0x142) at = row ? 16 * row - 1 : -1;
  else if (ctrl == 0x143) at = l >= 32 ? 31 : -1;
  else abort();
  if (at < 0 || !(row_mask >> row & 1)) return old;
  int v;
  memcpy(&v, all + 64 * at, sizeof v);
  return v;
}

void mfma_16x16x32_bf16(const void *x, const void *y, const float *c, float *d) {
  char both[32];
  memcpy(both, x, 16);
  memcpy(both + 16, y, 16);
  const char *all = static_cast<const char *>(exchange(both, sizeof both));
  const auto at = [&](int l, int which, int i) {
    uint16_t h;
    memcpy(&h, all + 64 * l + 16 * which + 2 * i, sizeof h);
    return (double)__builtin_bit_cast(float, (uint32_t)h << 16);
  };
  const int col = lane() % 16, quarter = lane() / 16;
  for (int r = 0; r < 4; ++r) {
    double s = c[r];
    for (int q = 0; q < 4; ++q)
      for (int i = 0; i < 8; ++i) s += at(16 * q + 4 * quarter + r, 0, i) * at(16 * q + col, 1, i);
    d[r] = (float)s;
  }
}

void launch(dim3 grid, dim3 block, const std::function<void()> &body) {
  const int n = (int)block.x;
  if (!stacks) stacks = static_cast<char *>(mmap(nullptr, kStack * 1024, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  grid_dim = grid;
  block_dim = block;
  work = &body;
  for (unsigned y = 0; y < grid.y; ++y)
    for (unsigned x = 0; x < grid.x; ++x) {
      block_idx = dim3(x, y);
      fibers.assign(n, Fiber());
      waves.assign((n + 63) / 64, Wave());
      if (hook) hook((int)(x + y * grid.x), -1);
      run_block(n);
    }
}
}  // namespace emu

// A call before a workgroup starts (barrier -1) and before each of its barriers lets go (nullptr: none), for tests that change memory meanwhile.
extern "C" void emu_set_hook(void (*h)(int block, int barrier)) { emu::hook = h; }
// x with lane `lane` replaced by the wave-uniform v.
extern "C" int emu_write_lane(int v, int lane, int x) __asm("llvm.amdgcn.writelane.i32");
extern "C" int emu_write_lane(int v, int lane, int x) { return emu::lane() == lane ? v : x; }

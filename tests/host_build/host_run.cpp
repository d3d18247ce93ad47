// Runs the workgroups of a launch one after the other, the threads of each as fibers; see hip/hip_runtime.h.
#include "hip/hip_runtime.h"

#include <cxxabi.h>
#include <dlfcn.h>
#include <signal.h>
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>
#include <unistd.h>

#include <map>
#include <set>
#include <string>
#include <vector>

// Saves the callee-saved registers and the stack of one fiber, goes on with another's.
extern "C" void host_switch(void** from, void* to);
asm(R"(
.globl host_switch
host_switch:
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

namespace host {
Fiber* current;
dim3 block, grid, block_size;
unsigned char* lds;

namespace {
enum { READY, IN_WAVE_OP, AT_BARRIER, DONE };
constexpr size_t kStack = 192 * 1024, kLds = 160 * 1024, kPage = 4096, kMaxThreads = 1024;
const char* kernel_name = "";
const std::function<void()>* kernel_body;
void* scheduler;
char* stacks;
unsigned char* lds_end;
size_t lds_size;
std::vector<Fiber> fibers(kMaxThreads);
std::map<const void*, int> lds_requests;  // dynamic LDS a kernel may be launched with, where more than 64 KB
std::set<std::string> launched;           // kernel instances so far, dynamic LDS and threads of a workgroup behind each
bool record_only;                         // note launches, run none
std::string only;                         // ... or run only kernels whose name holds this (empty: all)

void fail(const char* what, const void* at) {
  fprintf(stderr, "%s %p in %s, workgroup %u, %u of %u, %u, thread %u\n", what, at, kernel_name, block.x, block.y, grid.x, grid.y,
          current ? current->tid.x : 0);
  _exit(77);
}
void on_fault(int, siginfo_t* info, void*) { fail("access outside a buffer at", info->si_addr); }
void wait_in(int state) {
  Fiber* const me = current;
  me->state = state;
  host_switch(&me->sp, scheduler);
}
void fiber_main() {
  (*kernel_body)();
  wait_in(DONE);
}
char* map(size_t bytes) { return (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0); }

// Every lane that runs has come to a wave operation, a barrier or its end: the lanes in the operation exchange their values.
bool complete_wave_op(Fiber* wave, int lanes) {
  uint64_t active = 0, ballot = 0;
  for (int l = 0; l < lanes; ++l)
    if (wave[l].state == IN_WAVE_OP) {
      active |= 1ull << l;
      if (wave[l].kind == BALLOT && wave[l].value) ballot |= 1ull << l;
    }
  for (int l = 0; l < lanes; ++l)
    if (wave[l].state == IN_WAVE_OP) {
      Fiber& f = wave[l];
      const int from = f.kind == XOR ? l ^ f.arg : f.kind == UP ? l - f.arg : f.arg & 63;
      f.result = f.kind == BALLOT ? ballot : wave[from >= 0 && from < 64 && ((active >> from) & 1) ? from : l].value;
    }
  for (int l = 0; l < lanes; ++l)
    if (wave[l].state == IN_WAVE_OP) wave[l].state = READY;
  return active != 0;
}

void run_workgroup(int threads) {
  for (int t = 0; t < threads; ++t) {
    Fiber& f = fibers[t];
    f.state = READY;
    f.tid = dim3(t, 0, 0);
    f.lane = t & 63;
    void** sp = (void**)(stacks + kStack * (t + 1) - 64);
    *--sp = nullptr;
    *--sp = (void*)fiber_main;
    for (int i = 0; i < 6; ++i) *--sp = nullptr;
    f.sp = sp;
  }
  for (;;) {
    for (int w = 0; w < threads; w += 64) {
      const int lanes = std::min(64, threads - w);
      do {
        for (int t = w; t < w + lanes; ++t)
          if (fibers[t].state == READY) {
            current = &fibers[t];
            host_switch(&scheduler, current->sp);
          }
      } while (complete_wave_op(&fibers[w], lanes));
    }
    bool waiting = false;  // everyone is at the barrier or done
    for (int t = 0; t < threads; ++t)
      if (fibers[t].state == AT_BARRIER) {
        fibers[t].state = READY;
        waiting = true;
      }
    if (!waiting) return;
  }
}
}  // namespace

void barrier() { wait_in(AT_BARRIER); }
uint64_t wave_op(int kind, uint64_t value, int arg) {
  current->kind = kind;
  current->value = value;
  current->arg = arg;
  wait_in(IN_WAVE_OP);
  return current->result;
}

void request_lds(const void* function, int bytes) { lds_requests[function] = bytes; }
void launch(dim3 g, dim3 b, size_t lds_bytes, const char* kernel, const void* function, const std::function<void()>& body) {
  kernel_name = kernel;
  Dl_info info;
  if (dladdr(function, &info) && info.dli_sname && info.dli_saddr == function)
    if (char* const name = abi::__cxa_demangle(info.dli_sname, nullptr, nullptr, nullptr)) {
      launched.insert(std::string(name) + " lds " + std::to_string(lds_bytes) + " threads " + std::to_string(b.x));
      free(name);
    }
  kernel_body = &body;
  grid = g;
  block_size = b;
  if (lds_bytes > kLds || g.x == 0 || g.y == 0 || b.x > kMaxThreads) fail("launch bounds", nullptr);
  const auto request = lds_requests.find(function);
  if (lds_bytes > 64 * 1024 && (request == lds_requests.end() || (size_t)request->second < lds_bytes))
    fail("more dynamic LDS than requested:", (void*)lds_bytes);
  if (record_only || !strstr(kernel, only.c_str())) return;
  lds_size = (lds_bytes + 15) / 16 * 16;
  lds = lds_end - lds_size;
  for (unsigned y = 0; y < g.y; ++y)
    for (unsigned x = 0; x < g.x; ++x) {
      block = dim3(x, y, 0);
      run_workgroup((int)b.x);
    }
}

uint8_t load_byte(const Rsrc& r, unsigned voff, unsigned soff) {
  return (uint64_t)voff < r.bytes ? *reinterpret_cast<const volatile uint8_t*>(r.base + voff + soff) : 0;
}
unsigned load_dword(const Rsrc& r, unsigned voff, unsigned soff) {
  unsigned v = 0;
  if ((uint64_t)voff + 4 <= r.bytes) memcpy(&v, r.base + (size_t)voff + soff, 4);
  return v;
}
Chunk load_chunk(const Rsrc& r, unsigned voff, unsigned soff) {
  Chunk c = {0, 0, 0, 0};
  for (unsigned i = 0; i < 4; ++i)
    if ((uint64_t)voff + 4 * i < r.bytes) c[i] = load_dword(r, voff + 4 * i, soff);
  return c;
}
void store_chunk(const Chunk& c, const Rsrc& r, unsigned voff, unsigned soff) {
  for (unsigned i = 0; i < 4; ++i) {
    const unsigned v = c[i];
    if ((uint64_t)voff + 4 * i + 4 <= r.bytes) memcpy(const_cast<char*>(r.base) + (size_t)voff + 4 * i + soff, &v, 4);
  }
}
void load_to_lds(const Rsrc& r, unsigned voff, unsigned soff, unsigned lds_base) {
  const size_t at = lds_base + 16 * (size_t)current->lane;
  if (at + 16 > lds_size) fail("LDS-direct load past the launch's LDS at", (void*)at);
  const Chunk c = load_chunk(r, voff, soff);
  memcpy(lds + at, &c, 16);
}
void load_dword_to_lds(const Rsrc& r, unsigned voff, unsigned soff, unsigned lds_base) {
  const size_t at = lds_base + 4 * (size_t)current->lane;
  if (at + 4 > lds_size) fail("LDS-direct load past the launch's LDS at", (void*)at);
  const unsigned v = load_dword(r, voff, soff);
  memcpy(lds + at, &v, 4);
}
}  // namespace host

extern "C" void host_init() {
  using namespace host;
  stacks = map(kStack * kMaxThreads);
  char* const p = map(kLds + kPage);
  mprotect(p + kLds, kPage, PROT_NONE);
  lds_end = (unsigned char*)p + kLds;
  static char alt[65536];
  stack_t ss{};
  ss.ss_sp = alt;
  ss.ss_size = sizeof alt;
  sigaltstack(&ss, nullptr);
  struct sigaction sa{};
  sa.sa_sigaction = on_fault;
  sa.sa_flags = SA_SIGINFO | SA_ONSTACK;
  sigaction(SIGSEGV, &sa, nullptr);
  sigaction(SIGBUS, &sa, nullptr);
}

// A buffer with a page nobody may touch on either side; the buffer lies against the one behind it (16-byte aligned), or against
// the one ahead of it.
extern "C" void* host_alloc(size_t bytes, int front) {
  using namespace host;
  const size_t b = (bytes + 15) / 16 * 16, pages = (b + kPage - 1) / kPage * kPage;
  char* const p = map(pages + 2 * kPage);
  mprotect(p, kPage, PROT_NONE);
  mprotect(p + kPage + pages, kPage, PROT_NONE);
  return front ? p + kPage : p + kPage + pages - b;
}

// The kernel instances launched so far with the sizes of their workgroups, a line each; returns the bytes there are.
extern "C" size_t host_launched(char* out, size_t room) {
  std::string all;
  for (const std::string& k : host::launched) all += k + "\n";
  if (room > all.size()) memcpy(out, all.c_str(), all.size() + 1);
  return all.size();
}

// From now on launches are noted only: which kernels a call takes, at sizes that would run for long here.
extern "C" void host_record_only() { host::record_only = true; }

// From now on only launches of this kernel run: one kernel of a call whose others would run for long.
extern "C" void host_run_only(const char* kernel) { host::only = kernel; }

extern "C" int laud_probe_mfma() { return 0; }
extern "C" int laud_probe_read() { return 0; }
extern "C" int laud_probe_copy() { return 0; }

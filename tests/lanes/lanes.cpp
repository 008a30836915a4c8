// Runs the library's kernels on the CPU, lane by lane, and checks what a GPU would not tell: every access of a buffer resource or of
// a plain pointer lies in memory that the caller handed over, every LDS access in the LDS of its launch, lanes of a wavefront
// meet at the same exchange, wavefronts at the same barrier.
//
// A lane is a fiber.  A wavefront's lanes run one after the other up to the next point where they exchange something (a lane
// permutation, a matrix instruction, a transpose read), wavefronts one after the other up to the next barrier; blocks are dealt to a few
// host threads.  Loads from memory straight to LDS land either as they are issued ("early") or not before a wait forces them
// ("late"), and wavefronts and blocks run in ascending or descending order: a result that depends on a wait or a barrier that is
// not there differs between the two.
#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <cxxabi.h>
#include <dlfcn.h>
#include <atomic>
#include <cstdarg>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>

namespace lanes {
thread_local Idx tid, bid, bdim, gdim;
thread_local int lane;
static thread_local int wave;
static thread_local const void* kernel = nullptr;
static int late = 0;                       // loads to LDS land at their wait; wavefronts and blocks in descending order
static bool host_only = false;             // launches are looked at, not run
static std::atomic<long> complaints{0}, launches{0}, all_element_loads{0};
long launched() { return launches; }
thread_local long element_loads = 0;
static std::mutex mu;
static std::map<uintptr_t, size_t> ranges;      // device memory: start -> bytes (not changed while kernels run)

static std::string kernel_name(const void* k) {
    Dl_info d;
    if (!dladdr(k, &d) || !d.dli_sname) return "?";
    int st = 0;
    char* q = abi::__cxa_demangle(d.dli_sname, nullptr, nullptr, &st);
    std::string s = q ? q : d.dli_sname;
    free(q);
    return s.substr(0, s.find('('));
}
static void complain(const char* fmt, ...) {
    if (complaints++ >= 10) return;
    std::lock_guard<std::mutex> l(mu);
    va_list a;
    va_start(a, fmt);
    fprintf(stderr, "lanes: ");
    vfprintf(stderr, fmt, a);
    va_end(a);
    fprintf(stderr, " [block %u,%u,%u thread %u of %s]\n", bid.x, bid.y, bid.z, tid.x, kernel_name(kernel).c_str());
}

static bool owned(const void* p, size_t n) {
    auto it = ranges.upper_bound((uintptr_t)p);
    return it != ranges.begin() && (uintptr_t)p + n <= std::prev(it)->first + std::prev(it)->second;
}
static void check_owned(const void* p, size_t n, const char* what) {
    if (!owned(p, n)) complain("%s of %zu bytes outside every buffer", what, n);
}

// The bounds check of a raw buffer access: out of range where off >= records - soff.  Whether that difference wraps where soff
// is the larger one is nothing to rely on: only a lane that is masked (all ones) may come with such an soff.
bool in_buffer(const unsigned char* base, unsigned records, unsigned off, unsigned soff, unsigned bytes, bool store) {
    if (off == 0xffffffffu) return false;
    if (soff > records) {
        complain("buffer %s at %u relies on %u records - %u not wrapping", store ? "store" : "load", off, records, soff);
        return false;
    }
    if (off >= records - soff) return false;
    if ((uint64_t)off + bytes > records - soff) complain("buffer access of %u bytes at %u + %u straddles the end %u", bytes, off, soff, records);
    check_owned(base + off + soff, bytes, store ? "buffer store" : "buffer load");
    return true;
}

// ---- fibers --------------------------------------------------------------------------------------
extern "C" void lanes_switch(void** save, void* to);
asm(R"(
.text
.globl lanes_switch
lanes_switch:
    pushq %rbp; pushq %rbx; pushq %r12; pushq %r13; pushq %r14; pushq %r15
    movq %rsp, (%rdi)
    movq %rsi, %rsp
    popq %r15; popq %r14; popq %r13; popq %r12; popq %rbx; popq %rbp
    ret
)");

enum State { RUN, EXCHANGE, BARRIER, DONE };
struct Fiber {
    void* sp;
    char* stack;
    State state;
    int place;                 // source line it waits at
    unsigned exchanges, loads; // so far
};
struct Load { unsigned char* dst; unsigned char data[16]; };
constexpr size_t STACK = 128 * 1024;

struct Engine {
    std::vector<Fiber> f;
    void* main_sp = nullptr;
    int cur = -1;
    unsigned char *lds = nullptr, *map = nullptr;
    size_t lds_bytes = 0, map_bytes = 0;
    std::vector<std::vector<unsigned char>> slots;           // per wavefront two sets, used in turn
    std::vector<std::vector<std::vector<Load>>> loads;       // per wavefront and load to LDS: the lanes' parts
    const std::function<void()>* body = nullptr;

    ~Engine() {
        for (Fiber& x : f) munmap(x.stack, STACK);
        if (map) munmap(map, map_bytes);
    }
    // LDS between two pages without access, its end against the upper one
    void set_lds(size_t b) {
        const size_t pages = (b + 4095) / 4096 + (b == 0);
        map_bytes = (pages + 2) * 4096;
        map = (unsigned char*)mmap(nullptr, map_bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        mprotect(map, 4096, PROT_NONE);
        mprotect(map + (pages + 1) * 4096, 4096, PROT_NONE);
        lds = map + (pages + 1) * 4096 - ((b + 15) & ~(size_t)15);
        lds_bytes = b;
    }
};
static thread_local Engine* E = nullptr;

static void pause(State s, int place) {
    Fiber& x = E->f[E->cur];
    x.state = s;
    x.place = place;
    lanes_switch(&x.sp, E->main_sp);
}
static void fiber_main() {
    (*E->body)();
    pause(DONE, 0);
    abort();
}
static void resume(int i) {
    E->cur = i;
    tid = {(unsigned)i, 0, 0};
    lane = i & 63;
    wave = i >> 6;
    lanes_switch(&E->main_sp, E->f[i].sp);
}

void* dynamic_lds() { return E->lds; }
void barrier(int place) { pause(BARRIER, place); }
const unsigned char* exchange(const void* mine, size_t n, int place) {
    Fiber& x = E->f[E->cur];
    std::vector<unsigned char>& b = E->slots[(size_t)wave * 2 + (x.exchanges++ & 1)];
    b.resize(64 * 64);
    memcpy(b.data() + (size_t)lane * n, mine, n);
    pause(EXCHANGE, place);
    return b.data();
}

void load_to_lds(const unsigned* rsrc, unsigned char* dst, unsigned off, unsigned soff) {
    const unsigned char* base = (const unsigned char*)((uint64_t)rsrc[0] | ((uint64_t)rsrc[1] << 32));
    Load l{dst + lane * 16, {}};
    if (off != 0xffffffffu && (off & 3)) complain("load to LDS from misaligned offset %u", off);
    if (in_buffer(base, rsrc[2], off, soff, 16, false)) memcpy(l.data, base + off + soff, 16);
    if (l.dst < E->lds || l.dst + 16 > E->lds + E->lds_bytes) {
        complain("load to LDS at %ld of %zu bytes", (long)(l.dst - E->lds), E->lds_bytes);
        l.dst = nullptr;
    }
    auto& q = E->loads[wave];
    const unsigned k = E->f[E->cur].loads++;
    if (q.size() <= k) q.resize(k + 1);
    q[k].push_back(l);                     // (a wavefront's lanes come here in order)
    if (!late && l.dst) memcpy(l.dst, l.data, 16);
}
void wait_loads(int n) {
    const unsigned issued = E->f[E->cur].loads;
    if (!late || issued <= (unsigned)n) return;
    auto& q = E->loads[wave];
    for (unsigned k = 0; k < issued - n; ++k) {
        if ((int)q[k].size() <= lane || !q[k][lane].dst) continue;
        memcpy(q[k][lane].dst, q[k][lane].data, 16);
        q[k][lane].dst = nullptr;
    }
}

static void run_block(int n) {
    const int waves = (n + 63) / 64;
    E->slots.resize((size_t)waves * 2);
    E->loads.assign(waves, {});
    while ((int)E->f.size() < n) {
        Fiber x{};
        x.stack = (char*)mmap(nullptr, STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        E->f.push_back(x);
    }
    for (int i = 0; i < n; ++i) {
        Fiber& x = E->f[i];
        void** sp = (void**)(x.stack + STACK - 64);
        *--sp = nullptr;
        *--sp = (void*)fiber_main;
        for (int k = 0; k < 6; ++k) *--sp = nullptr;
        x = Fiber{sp, x.stack, RUN, 0, 0, 0};
    }
    memset(E->lds, 0xCB, E->lds_bytes);
    for (;;) {
        for (int k = 0; k < waves; ++k) {
            const int w = late ? waves - 1 - k : k, a = w * 64, b = std::min(n, a + 64);
            for (;;) {
                for (int i = a; i < b; ++i) if (E->f[i].state == RUN) resume(i);
                int waiting = 0, blocked = 0, place = 0;
                for (int i = a; i < b; ++i) {
                    if (E->f[i].state == BARRIER) ++blocked;
                    if (E->f[i].state != EXCHANGE) continue;
                    if (waiting++ && E->f[i].place != place) { complain("lanes of a wavefront wait at lines %d and %d", place, E->f[i].place); exit(3); }
                    place = E->f[i].place;
                }
                if (!waiting) break;
                if (blocked) { complain("some lanes of a wavefront wait at line %d, others at a barrier", place); exit(3); }
                for (int i = a; i < b; ++i) if (E->f[i].state == EXCHANGE) E->f[i].state = RUN;
            }
        }
        int place = -1, left = 0;
        for (int i = 0; i < n; ++i) {
            if (E->f[i].state == DONE) continue;
            ++left;
            if (place >= 0 && E->f[i].place != place) complain("barriers at lines %d and %d", place, E->f[i].place);
            place = E->f[i].place;
            E->f[i].state = RUN;
        }
        if (!left) break;
    }
    for (auto& q : E->loads) for (auto& l : q) if (l.size() != 64) complain("a load to LDS by %zu lanes", l.size());
}

// ---- launches ------------------------------------------------------------------------------------
static thread_local int current_device = 0;
static std::set<std::pair<int, const void*>> lds_allowed;      // devices and kernels that may have more than 64 KB of LDS
int device() { return current_device; }
int set_device(int d) { current_device = d; return hipSuccess; }
int allow_lds(const void* k, int) {
    std::lock_guard<std::mutex> l(mu);
    lds_allowed.insert({current_device, k});
    return hipSuccess;
}

void run(dim3 grid, dim3 block, size_t lds, const void* k, const std::function<void()>& body) {
    const int64_t blocks = (int64_t)grid.x * grid.y * grid.z;
    const int threads = (int)(block.x * block.y * block.z);
    static const bool trace = getenv("LPM_LANES_TRACE") != nullptr;
    kernel = k;
    ++launches;
    if (trace) fprintf(stderr, "lanes: %ux%ux%u blocks of %d threads, %zu bytes of LDS: %s\n", grid.x, grid.y, grid.z, threads, lds, kernel_name(k).c_str());
    bool allowed = lds <= 64 * 1024;
    if (!allowed) {
        std::lock_guard<std::mutex> l(mu);
        allowed = lds_allowed.count({current_device, k}) != 0;
    }
    if (blocks <= 0 || threads <= 0 || threads > 1024 || lds > 160 * 1024 || !allowed) {
        complain("a launch of %lld blocks of %d threads with %zu bytes of LDS that device %d does not take", (long long)blocks, threads, lds, current_device);
        return;
    }
    if (host_only) return;
    std::atomic<int64_t> next{0};
    auto work = [&]() {
        Engine e;
        E = &e;
        kernel = k;
        e.set_lds(lds);
        e.body = &body;
        bdim = {block.x, block.y, block.z};
        gdim = {grid.x, grid.y, grid.z};
        for (int64_t k; (k = next++) < blocks;) {
            const int64_t i = late ? blocks - 1 - k : k;
            bid = {(unsigned)(i % grid.x), (unsigned)(i / grid.x % grid.y), (unsigned)(i / ((int64_t)grid.x * grid.y))};
            run_block(threads);
        }
        all_element_loads += element_loads;      // (a thread serves one launch)
    };
    std::vector<std::thread> pool;
    for (int64_t i = 0; i < std::min<int64_t>(8, blocks); ++i) pool.emplace_back(work);
    for (std::thread& t : pool) t.join();
}
}  // namespace lanes

extern "C" {
// n bytes of device memory: between pages without access, their end (on a multiple of 256 bytes) against the upper one.  It is never
// given back, so no address means two things in one process.
void* lanes_alloc(size_t n) {
    const size_t pages = (n + 4095) / 4096 + (n == 0), guard = 4 * 4096;
    unsigned char* m = (unsigned char*)mmap(nullptr, pages * 4096 + 2 * guard, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    mprotect(m, guard, PROT_NONE);
    mprotect(m + guard + pages * 4096, guard, PROT_NONE);
    unsigned char* p = m + guard + pages * 4096 - ((n + 255) & ~(size_t)255);
    if (n) lanes::ranges[(uintptr_t)p] = n;
    return p;
}
// whether n bytes from p are device memory, in one allocation
int lanes_owned(const void* p, size_t n) { return lanes::owned(p, n); }
void lanes_late(int v) { lanes::late = v; }
void lanes_host_only(int v) { lanes::host_only = v != 0; }
void lanes_set_device(int d) { lanes::set_device(d); }
long lanes_complaints() { return lanes::complaints; }
long lanes_element_loads() { return lanes::all_element_loads; }
}

// Runtime of the CPU emulation: a pool of OS threads, as many as the largest block so far had, plays the threads of one block;
// blocks of a launch run one after another.
#include <hip/hip_runtime.h>

#include <chrono>
#include <climits>
#include <execinfo.h>
#include <linux/futex.h>
#include <mutex>
#include <sched.h>
#include <signal.h>
#include <sys/mman.h>
#include <sys/syscall.h>
#include <thread>
#include <unistd.h>
#include <vector>

thread_local dim3 threadIdx, blockIdx;
dim3 blockDim, gridDim;
thread_local const char* emu_where = "";
thread_local int emu_line = 0;
alignas(64) static char g_lds[160 * 1024];
char* emu_dyn_lds = g_lds;
extern "C" { int emu_last_error = 0, emu_fail_launch = 0, emu_host_blocks = 0; }

constexpr int MAXT = 1024;
static thread_local int t_id = -1;   // index in the pool, -1: host thread
static const char* g_where[MAXT];
static int g_wline[MAXT];
static int g_block = 0;
static const char* g_kernel = "";

static void dump_all(const char* why) {
    fprintf(stderr, "\n[emu] %s; block %d of %u, blockDim %u\n", why, g_block, gridDim.x, blockDim.x);
    for (unsigned t = 0; t < blockDim.x && t < MAXT; ++t)
        if (t < 8 || t % 64 == 0 || t % 64 == 63 || g_wline[t] != g_wline[0])
            fprintf(stderr, "  thread %3u last at %s:%d\n", t, g_where[t] ? g_where[t] : "?", g_wline[t]);
    fflush(stderr);
}
static void note() {
    if (t_id >= 0) { g_where[t_id] = emu_where; g_wline[t_id] = emu_line; }
}

// Arrivals and members in one word, so that a thread that leaves and one that arrives cannot both miss that everyone is there; waiters sleep on the
// generation (a condition variable would have every woken thread queue for its mutex: four times the time of a launch).
struct Barrier {
    std::atomic<uint64_t> state{0};   // members << 32 | arrived
    std::atomic<uint32_t> gen{0};
    void init(int n) { state = (uint64_t)n << 32; }
    void grow(int n) {   // while the launching thread is not waiting: nobody is released
        uint64_t s = state;
        while (!state.compare_exchange_weak(s, (uint64_t)n << 32 | (uint32_t)s)) {}
    }
    void release() {
        ++gen;
        syscall(SYS_futex, &gen, FUTEX_WAKE_PRIVATE, INT_MAX, nullptr, nullptr, 0);
    }
    void wait(const char* what) {
        note();
        const uint32_t g = gen;
        uint64_t s = state, next;
        do next = (uint32_t)s + 1 >= s >> 32 ? s >> 32 << 32 : s + 1;
        while (!state.compare_exchange_weak(s, next));
        if (!(uint32_t)next) { release(); return; }
        // the idle pool waits for ever, and the launching thread for the whole launch: long for a large case, and a hang inside it is reported by the
        // workers' own waits.  Any other wait that outlasts the limit is taken for a deadlock (EMU_WAIT_SECONDS raises it).
        const bool for_ever = (what[0] == 's' && what[1] == 't') || (what[0] == 'd' && what[1] == 'o');
        static const int limit = getenv("EMU_WAIT_SECONDS") ? atoi(getenv("EMU_WAIT_SECONDS")) : 60;
        const auto until = std::chrono::steady_clock::now() + std::chrono::seconds(limit);
        while (gen == g) {
            const timespec second{1, 0};
            syscall(SYS_futex, &gen, FUTEX_WAIT_PRIVATE, g, for_ever ? nullptr : &second, nullptr, 0);
            if (!for_ever && gen == g && std::chrono::steady_clock::now() > until) {
                fprintf(stderr, "[emu] barrier '%s' timed out: %d of %d arrived (thread %d)\n", what, (int)(uint32_t)state, (int)(state >> 32), t_id);
                dump_all("deadlock");
                abort();
            }
        }
    }
    // a thread that leaves the kernel no longer takes part in __syncthreads
    void leave() {
        uint64_t s = state, next;
        do {
            next = s - (1ull << 32);
            if (next >> 32 && (uint32_t)next >= next >> 32) next = next >> 32 << 32;
        } while (!state.compare_exchange_weak(s, next));
        if ((uint32_t)s && !(uint32_t)next) release();
    }
};

static Barrier &b_start = *new Barrier, &b_done = *new Barrier, &b_blk = *new Barrier, &b_sync = *new Barrier;
static Barrier* const b_wave = new Barrier[MAXT / 64];   // never destroyed: idle workers sleep on them at exit
static std::function<void()> g_body;
static int g_nthreads = 0;
static std::vector<std::thread>& g_pool = *new std::vector<std::thread>;
static std::atomic<long long> g_clock{0};

static void on_segv(int sig, siginfo_t* si, void*) {
    fprintf(stderr, "\n[emu] signal %d at address %p: block %u thread %u (pool %d), last collective %s:%d\n", sig,
            si->si_addr, blockIdx.x, threadIdx.x, t_id, emu_where, emu_line);
    void* bt[48];
    const int n = backtrace(bt, 48);
    backtrace_symbols_fd(bt, n, 2);
    _exit(139);
}

static void worker(int id) {
    t_id = id;
    for (;;) {
        b_start.wait("start");
        if (id < g_nthreads) {
            for (unsigned blk = 0; blk < gridDim.x * gridDim.y * gridDim.z; ++blk) {
                blockIdx = dim3(blk % gridDim.x, (blk / gridDim.x) % gridDim.y, blk / (gridDim.x * gridDim.y));
                threadIdx = dim3(id % blockDim.x, (id / blockDim.x) % blockDim.y, id / (blockDim.x * blockDim.y));
                if (id == 0) { g_block = (int)blk; b_sync.init(g_nthreads); }
                b_blk.wait("block begin");
                g_body();
                b_sync.leave();
                b_blk.wait("block end");
            }
        }
        b_done.wait("done");
    }
}

void emu_launch(const std::function<void()>& body, dim3 grid, dim3 block, size_t shmem) {
    static bool once = false;
    if (!once) {
        once = true;
        struct sigaction sa;
        memset(&sa, 0, sizeof sa);
        sa.sa_sigaction = on_segv;
        sa.sa_flags = SA_SIGINFO;
        sigaction(SIGSEGV, &sa, nullptr);
        sigaction(SIGBUS, &sa, nullptr);
    }
    const int nt = (int)(block.x * block.y * block.z);
    if (nt > MAXT || nt % 64) { fprintf(stderr, "[emu] unsupported block size %d\n", nt); abort(); }
    if (shmem > sizeof g_lds) { fprintf(stderr, "[emu] dynamic LDS too large\n"); abort(); }
    if (grid.x * grid.y * grid.z == 0) return;
    if ((int)g_pool.size() < nt) {   // (idle workers take part in every launch's start and end: no more of them than needed)
        b_start.grow(nt + 1);
        b_done.grow(nt + 1);
        while ((int)g_pool.size() < nt) { g_pool.emplace_back(worker, (int)g_pool.size()); g_pool.back().detach(); }
    }
    g_body = body;
    gridDim = grid;
    blockDim = block;
    g_nthreads = nt;
    b_blk.init(nt);
    b_sync.init(nt);
    for (int w = 0; w < MAXT / 64; ++w) b_wave[w].init(64);
    b_start.wait("start");
    b_done.wait("done");
}

// ---- what is touched ahead ----
extern "C" { int emu_logging = 0; }
struct Event { uint64_t launch, what, address, x, y; };   // what: 0 a touched line by workgroup x, 1 a linear map (x: bytes to the next of y maps)
static std::mutex& g_events_lock = *new std::mutex;
static std::vector<Event>& g_events = *new std::vector<Event>;
static uint64_t g_launch = 0;
void emu_log_launch() { ++g_launch; }
void emu_log_map(const void* weights, size_t stride, unsigned maps) { g_events.push_back({g_launch, 1, (uint64_t)weights, stride, maps}); }
uint32_t emu_touch_load(const uint32_t* p) {
    const uint32_t v = *(const volatile uint32_t*)p;
    if (emu_logging) {
        std::lock_guard<std::mutex> lk(g_events_lock);
        g_events.push_back({g_launch, 0, (uint64_t)p, blockIdx.x, blockIdx.y});
    }
    return v;
}
// Takes the events since the last call, oldest first, five words each; returns how many there are.
extern "C" size_t emu_take_events(uint64_t* out, size_t room) {
    const size_t n = g_events.size();
    if (!out) return n;
    memcpy(out, g_events.data(), std::min(n, room) * sizeof(Event));
    g_events.clear();
    return n;
}

void emu_syncthreads() { b_sync.wait("__syncthreads"); }
void emu_yield() { sched_yield(); }
long long emu_clock() { return ++g_clock; }

// ---- pairwise exchange for __shfl_xor ----
struct Slot {
    std::atomic<uint64_t> seq[8];
    uint64_t cnt[8];
    uint32_t val[8][4];
};
static Slot g_slot[MAXT];

uint32_t emu_shfl_xor32(uint32_t v, int mask) {
    // one exchange channel per mask: the powers of two, and 7 / 15 (the mirrored half row / row of the
    // DPP permutations, which are the exchanges i <-> i ^ 7 and i <-> i ^ 15)
    const bool pow2 = mask > 0 && mask < 64 && !(mask & (mask - 1));
    if (!pow2 && mask != 7 && mask != 15) { fprintf(stderr, "[emu] shfl_xor mask %d\n", mask); abort(); }
    const int bit = pow2 ? __builtin_ctz(mask) : mask == 7 ? 6 : 7, me = t_id, other = me ^ mask;
    Slot& a = g_slot[me];
    Slot& b = g_slot[other];
    const uint64_t k = a.cnt[bit]++;
    a.val[bit][k & 3] = v;
    a.seq[bit].store(k + 1, std::memory_order_release);
    note();
    long spins = 0;
    while (b.seq[bit].load(std::memory_order_acquire) < k + 1) {
        sched_yield();
        if (++spins > 20000000) {
            fprintf(stderr, "[emu] shfl_xor(%d): lane %d waits for lane %d that never came (%s:%d)\n", mask, me, other,
                    emu_where, emu_line);
            dump_all("divergent shuffle");
            abort();
        }
    }
    return b.val[bit][k & 3];
}

static uint32_t g_xch[MAXT];
uint32_t emu_shfl_down32(uint32_t v, int delta) {
    const int me = t_id, w = me >> 6, lane = me & 63;
    g_xch[me] = v;
    b_wave[w].wait("shfl_down");
    const uint32_t r = lane + delta < 64 ? g_xch[me + delta] : v;
    b_wave[w].wait("shfl_down");
    return r;
}

uint32_t emu_shfl_idx32(uint32_t v, int src) {
    const int me = t_id, w = me >> 6;
    g_xch[me] = v;
    b_wave[w].wait("shfl");
    const uint32_t r = g_xch[(w << 6) + (src & 63)];
    b_wave[w].wait("shfl");
    return r;
}

int emu_all(int pred) {
    const int me = t_id, w = me >> 6;
    g_xch[me] = pred ? 1 : 0;
    b_wave[w].wait("all");
    int r = 1;
    for (int i = 0; i < 64; ++i) r &= (int)g_xch[(w << 6) + i];
    b_wave[w].wait("all");
    return r;
}

static uint16_t g_a[MAXT][8], g_b[MAXT][8];
static inline float bf(uint16_t x) { uint32_t u = (uint32_t)x << 16; float f; memcpy(&f, &u, 4); return f; }
void emu_mfma_16x16x32_bf16(const uint16_t a[8], const uint16_t b[8], float c[4]) {
    const int me = t_id, w = me >> 6, lane = me & 63, base = w * 64;
    memcpy(g_a[me], a, 16);
    memcpy(g_b[me], b, 16);
    b_wave[w].wait("mfma");
    const int col = lane & 15;
    for (int i = 0; i < 4; ++i) {
        const int row = 4 * (lane >> 4) + i;
        float acc = 0.f;
        for (int k = 0; k < 32; ++k)
            acc += bf(g_a[base + row + 16 * (k >> 3)][k & 7]) * bf(g_b[base + col + 16 * (k >> 3)][k & 7]);
        c[i] += acc;
    }
    b_wave[w].wait("mfma");
}

// Arena with inaccessible pages on both sides; the usable range ends right at the upper guard.
extern "C" void* emu_alloc(size_t n, int fill) {
    const size_t pg = 4096, body = (n + 255) / 256 * 256, span = (body + pg - 1) / pg * pg;
    char* p = (char*)mmap(nullptr, span + 2 * pg, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    mprotect(p, pg, PROT_NONE);
    mprotect(p + pg + span, pg, PROT_NONE);
    char* base = p + pg + (span - body);
    memset(p + pg, fill, span);
    return base;
}

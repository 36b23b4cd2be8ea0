// Runs kernels on the CPU, a workgroup at a time, every lane a fibre.  Memory lies next to pages that may not be touched, so
// that plain pointers are checked too: such an access ends the process, others are counted and printed.
#include <hip/hip_runtime.h>
#include <signal.h>
#include <sys/mman.h>
#include <ucontext.h>
#include <unistd.h>
#include <map>

namespace lanes {
Lane *now;
namespace {
constexpr size_t kStack = 256 * 1024, kPage = 4096;
struct Fibre {
    ucontext_t context;
    Lane lane;
    bool done;
};
struct Meeting {
    int here = 0;
    uint64_t round = 0, in[64], out[64];
};
std::vector<Fibre> fibres;
std::vector<unsigned char *> stacks;
std::vector<Meeting> waves, rows;
Meeting group;
ucontext_t scheduler;
size_t running, alive;
std::function<void()> kernel_now;
const char *name_now = "";
uintptr_t lds_at;
size_t lds_bytes_now;
std::map<uintptr_t, size_t> allocations;
long n_reports;

void yield()
{
    const size_t me = running;
    swapcontext(&fibres[me].context, &scheduler);
    now = &fibres[me].lane;
}

const uint64_t *meet(Meeting &m, int of, int place, uint64_t v)
{
    m.in[place] = v;
    const uint64_t round = m.round;
    if (++m.here == of) {
        memcpy(m.out, m.in, sizeof m.out);
        m.here = 0;
        m.round++;
    } else {
        while (m.round == round) yield();
    }
    return m.out;
}

void run_fibre()
{
    kernel_now();
    fibres[running].done = true;
    alive--;
    swapcontext(&fibres[running].context, &scheduler);
}

unsigned char *fenced(size_t bytes, size_t &pages)
{
    pages = (bytes + kPage - 1) / kPage * kPage;
    unsigned char *m = static_cast<unsigned char *>(mmap(nullptr, pages + 2 * kPage, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    mprotect(m + kPage, pages, PROT_READ | PROT_WRITE);
    return m + kPage;
}

void on_fault(int, siginfo_t *info, void *)
{
    char text[256];
    const int n = snprintf(text, sizeof text, "OUT OF RANGE %s: address %p, workgroup %u, lane %u\n", name_now, info->si_addr,
                           now ? now->bid.x : 0u, now ? now->tid.x : 0u);
    if (write(1, text, (size_t)n) < 0) {}
    _exit(3);
}
struct Handler {
    Handler()
    {
        static unsigned char stack[65536];
        stack_t s{};
        s.ss_sp = stack;
        s.ss_size = sizeof stack;
        sigaltstack(&s, nullptr);
        struct sigaction a {};
        a.sa_sigaction = on_fault;
        a.sa_flags = SA_SIGINFO | SA_ONSTACK;
        sigaction(SIGSEGV, &a, nullptr);
    }
} handler;
}  // namespace

uintptr_t lds_base() { return lds_at; }
size_t lds_size() { return lds_bytes_now; }
const uint64_t *wave_values(uint64_t v) { return meet(waves[now->tid.x >> 6], 64, lane(), v); }
const uint64_t *row_values(uint64_t v) { return meet(rows[now->tid.x >> 4], 16, lane(), v); }
void barrier() { meet(group, (int)now->bdim.x, 0, 0); }

bool inside(uintptr_t at, size_t n)
{
    auto it = allocations.upper_bound(at);
    if (it == allocations.begin()) return false;
    --it;
    return at + n <= it->first + it->second;
}

void report(const char *what, uintptr_t at, size_t n)
{
    if (n_reports++ < 8)
        printf("OUT OF RANGE %s: %zu bytes of %s at %#zx (%zu of LDS), workgroup %u, lane %u\n", name_now, n, what, (size_t)at, lds_bytes_now,
               now->bid.x, now->tid.x);
    fflush(stdout);
}

void launch(std::function<void()> kernel, dim3 grid, dim3 block, size_t lds_bytes, const char *name)
{
    const size_t n = block.x;
    if (n % 64) abort();
    name_now = name;
    kernel_now = std::move(kernel);
    while (stacks.size() < n)
        stacks.push_back(static_cast<unsigned char *>(mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0)));
    size_t pages;
    lds_bytes_now = (lds_bytes + 15) / 16 * 16;
    unsigned char *m = fenced(lds_bytes_now + 16, pages);
    lds_at = reinterpret_cast<uintptr_t>(m) + pages - lds_bytes_now;
    for (unsigned b = 0; b < grid.x; b++) {
        memset(lds(), 0xA5, lds_bytes_now);
        fibres = std::vector<Fibre>(n);
        waves.assign(n / 64, Meeting());
        rows.assign(n / 16, Meeting());
        group = Meeting();
        alive = n;
        for (size_t i = 0; i < n; i++) {
            Fibre &f = fibres[i];
            getcontext(&f.context);
            f.context.uc_stack.ss_sp = stacks[i];
            f.context.uc_stack.ss_size = kStack;
            f.context.uc_link = nullptr;
            f.lane = Lane{dim3((unsigned)i, 0, 0), dim3(b, 0, 0), block, grid};
            f.done = false;
            makecontext(&f.context, run_fibre, 0);
        }
        while (alive)
            for (size_t i = 0; i < n; i++) {
                if (fibres[i].done) continue;
                running = i;
                now = &fibres[i].lane;
                swapcontext(&scheduler, &fibres[i].context);
            }
    }
    munmap(m - kPage, pages + 2 * kPage);
}

int compute_units()
{
    static const int n = std::getenv("LANES_COMPUTE_UNITS") ? std::atoi(std::getenv("LANES_COMPUTE_UNITS")) : 6;
    return n;
}
}  // namespace lanes

extern "C" {
// `bytes` of "device" memory, its end (at_start: its start) next to a page that may not be touched
void *lanes_alloc(size_t bytes, int at_start, size_t align)
{
    size_t pages;
    bytes = std::max<size_t>(1, (bytes + align - 1) / align) * align;
    unsigned char *m = lanes::fenced(bytes, pages);
    unsigned char *p = at_start ? m : m + pages - bytes;
    lanes::allocations[reinterpret_cast<uintptr_t>(p)] = bytes;
    return p;
}
long lanes_reports() { return lanes::n_reports; }
}

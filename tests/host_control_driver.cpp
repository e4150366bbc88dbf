// Checks of the parts of the CG's control that host and device code share, run
// on the host by tests/test_host_control.py: `host_control_driver CHECK`
// returns 0 when the check named holds. Nothing here reaches a GPU.
#include "../paper_1908_03301_amd/csrc/rn_cg.hpp"

#include <cstdio>
#include <cstring>

using namespace rn;

namespace {

int fails = 0;

void expect(bool ok, const char *what)
{
    if (!ok) {
        std::fprintf(stderr, "unexpected: %s\n", what);
        ++fails;
    }
}

// A workgroup that gives up a wait raises loop_failed in memory. Workgroup 0
// took its copy of the control block before and may reach its end regardless:
// what it stores must leave the flag standing, and everything else new.
void loop_end_keeps_failure()
{
    Scalars mem, copy;
    std::memset(&mem, 0, sizeof(mem));
    mem.iters = 5;
    copy = mem;                       // at the start of the loop
    copy.iters = 90;                  // ... its steps
    copy.mode = MODE_REFRESH;
    copy.xr = 2.5;
    mem.loop_failed = 1;              // another workgroup, meanwhile
    mem.loop_aborts = 3;
    unsigned long long words[kScalWords], own[kScalWords];
    std::memcpy(words, &mem, sizeof(mem));
    std::memcpy(own, &copy, sizeof(copy));
    for (int t = 0; t < kBlock; ++t) store_loop_end(words, own, t);
    std::memcpy(&mem, words, sizeof(mem));
    expect(mem.loop_failed == 1u, "the failure flag is erased");
    expect(mem.loop_aborts == 3u, "the count of refusals is erased");
    expect(mem.iters == 90 && mem.mode == MODE_REFRESH && mem.xr == 2.5, "the loop's own state is not stored");
}

}  // namespace

int main(int argc, char **argv)
{
    const char *want = argc > 1 ? argv[1] : "";
    if (!std::strcmp(want, "loop_end_keeps_failure")) loop_end_keeps_failure();
    else expect(false, "no such check");
    std::printf("%s: %d failures\n", want, fails);
    return fails != 0;
}

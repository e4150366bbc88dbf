// Checks of the parts of the CG's control that host and device code share, run
// on the host by tests/test_host_control.py: `host_control_driver CHECK`
// returns 0 when the check named holds. Nothing here reaches a GPU.
#include "../paper_1908_03301_amd/csrc/rn_cg.hpp"

#include <cmath>
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

// The scalar step of the pass kernels and of the resident loops have to give
// the same bits whatever the compiler makes of a sum of products: r.z of the
// next pass is two fused operations, on a host that fuses none by itself.
void step_rounds_as_written()
{
    unsigned long long h = 88172645463325252ull;
    auto uniform = [&] {
        h ^= h << 13;
        h ^= h >> 7;
        h ^= h << 17;
        return 0.5 + (double)(h >> 11) * 0x1p-53;
    };
    int wrong = 0;
    for (int k = 0; k < 1000; ++k) {
        const double rz = uniform(), pq = 2.0 * uniform(), zq = 0.3 * uniform(), qq = 4.0 * uniform();
        const double t[kRed] = {pq, zq, qq, rz, 0.0};
        Scalars s;
        std::memset(&s, 0, sizeof(s));
        s.sigma = s.kappa = s.bhat = 1.0;
        s.max_iter = 1000;
        s.kpend = 4;
        step_after_cg(&s, t);
        const double alpha = rz / pq, next = std::fma(alpha * alpha, qq, std::fma(-2.0 * alpha, zq, rz));
        if (!(next > 0.0)) continue;
        wrong += s.mode != MODE_CG || s.alpha != alpha || s.beta != next / rz || s.est_rel != std::sqrt(next);
    }
    expect(wrong == 0, "a step with another rounding");
}

// The indices of a thread of a launch, also where n is within a stride of 2^31
// (nodes) or 2^32 (positions of a tour).
template <bool FAR>
void strided(unsigned long long n)
{
    for (unsigned step : {256u, 2097152u}) {
        if (n > 10000000ull && step == 256u) continue;
        for (unsigned first : {0u, 1u, step / 2, step - 1}) {
            const unsigned long long expected = n > first ? (n - first + step - 1) / step : 0;
            unsigned long long count = 0, next = first;
            bool inside = true;
            for (const unsigned i : Strided<FAR>{{first, step, (unsigned)n}}) {
                inside = inside && i == next && i < n;
                next += step;
                if (++count > expected) break;
            }
            expect(inside && count == expected, "indices of a thread");
        }
    }
}

void strides_end()
{
    for (unsigned long long n : {0ull, 1ull, 255ull, 256ull, 257ull, 1000ull, 5ull << 20, 2147483645ull}) {
        strided<false>(n);
        strided<true>(n);
    }
    for (unsigned long long n : {4294605841ull, 4294967295ull}) strided<true>(n);
}

}  // namespace

int main(int argc, char **argv)
{
    const char *want = argc > 1 ? argv[1] : "";
    if (!std::strcmp(want, "loop_end_keeps_failure")) loop_end_keeps_failure();
    else if (!std::strcmp(want, "step_rounds_as_written")) step_rounds_as_written();
    else if (!std::strcmp(want, "strides_end")) strides_end();
    else expect(false, "no such check");
    std::printf("%s: %d failures\n", want, fails);
    return fails != 0;
}

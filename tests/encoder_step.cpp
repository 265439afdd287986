// Checks the encoder's renormalisation and its step that codes nothing on the host: the same function and constants as the
// kernel's, every frequency and the states around every limit.  Prints "ok" or what is wrong.
#include <cstdint>
#include <cstdio>
#include "neuzip_format.h"

namespace {

uint64_t g_checked = 0;

// x after the step of constants e, as EncSym states it; a word pushed in front of it says so
uint32_t step(uint32_t x, const nz::EncSym &e, bool &pushed)
{
    pushed = nz::renormalises(x, e.limit_cum);
    if (pushed)
        x >>= 16;
    const uint32_t inc_x = x + (e.shift_inc >> 16);
    const uint32_t q = static_cast<uint32_t>((static_cast<uint64_t>(inc_x) * e.mul) >> 32) >> (e.shift_inc & 31u);
    return (q & 0xFFFFFFu) * (e.cmpl & 0xFFFFFFu) + x + (e.limit_cum & 0xFFFFu);
}

bool leaves_as_it_is(uint64_t state)
{
    const uint32_t x = static_cast<uint32_t>(state);
    bool pushed = false;
    ++g_checked;
    if (step(x, nz::kNoSymbol, pushed) == x && !pushed)
        return true;
    std::printf("no symbol: state %08x is left as %08x, a word pushed: %d\n", x, step(x, nz::kNoSymbol, pushed), pushed);
    return false;
}

}  // namespace

int main()
{
    constexpr uint64_t kLow = nz::kRansL, kEnd = 1ull << 32, kReach = 70000;
    // the step that codes nothing, over both ends of the interval and between
    for (uint64_t x = kLow; x < kLow + kReach; ++x)
        if (!leaves_as_it_is(x))
            return 1;
    for (uint64_t x = kEnd - kReach; x < kEnd; ++x)
        if (!leaves_as_it_is(x))
            return 1;
    for (uint64_t x = kLow; x < kEnd; x += 65521)
        if (!leaves_as_it_is(x))
            return 1;
    // every frequency: renormalised from f * 2^20 on, never where f is the whole table or nothing
    for (uint64_t f = 0; f <= nz::kM; ++f) {
        const uint64_t limit = f << 20;
        for (uint32_t cum : {0u, 1u, 4095u}) {
            const uint32_t limit_cum = nz::limit_of(static_cast<uint32_t>(f)) | cum;
            if ((limit_cum & 0xFFFFu) != cum)
                return std::printf("f = %u: cum does not fit beside the limit\n", static_cast<unsigned>(f)), 1;
            for (uint64_t base : {limit, kLow + 4, kEnd - 4, static_cast<uint64_t>(0xFFFF0000u)})
                for (uint64_t x = base >= kLow + 4 ? base - 4 : kLow; x < base + 4 && x < kEnd; ++x, ++g_checked)
                    if (nz::renormalises(static_cast<uint32_t>(x), limit_cum) != (f > 0 && x >= limit))
                        return std::printf("f = %u: state %08x\n", static_cast<unsigned>(f), static_cast<unsigned>(x)), 1;
        }
    }
    std::printf("%llu states ok\n", static_cast<unsigned long long>(g_checked));
    return 0;
}

"""Arithmetic that the kernels share with the host (csrc/arith.h), on the CPU: a program with the header's own code, built with the host compiler."""
import pytest

from _util import run_host_program


@pytest.mark.parametrize("seed", range(4))
def test_arrivals_of_overlapping_calls_leave_no_count_behind(tmp_path, seed):
    """Calls with any numbers of heads and parts whose blocks arrive in any order, mixed with those of other calls: when all have
    arrived every counter is at zero, and a call by itself has one last block a head, the one that arrives last."""
    run_host_program(tmp_path, """
int main() {
    srand(%d);
    std::vector<uint32_t> counters(64 * kAttnPartials);
    auto arrive = [&](int head, int parts) {
        uint32_t& c = counters[arrival_counter(head, parts)];
        const uint32_t before = c;
        c = before >= (uint32_t)parts - 1u ? 0u : before + 1u;         // what atomicInc(&c, parts - 1) does
        return last_arrival(before, parts);
    };
    struct Block { int head, parts; };
    for (int round = 0; round < 400; ++round) {
        std::vector<Block> blocks;
        for (int calls = rand() %% 4 + 2; calls > 0; --calls) {
            const int heads = rand() %% 64 + 1, parts = rand() %% 3 ? rand() %% 20 + 2 : rand() %% 255 + 2;
            for (int b = 0; b < heads * parts; ++b) blocks.push_back({b %% heads, parts});
        }
        for (size_t i = blocks.size(); i > 1; --i) std::swap(blocks[i - 1], blocks[rand() %% i]);
        for (const Block& b : blocks) arrive(b.head, b.parts);
        for (uint32_t c : counters)
            if (c != 0) { printf("round %%d: a counter is left at %%u\\n", round, c); return 1; }
        const int parts = rand() %% 256 + 1;
        for (int head = 0; head < 64; ++head)
            for (int k = 0; k < parts; ++k)
                if (arrive(head, parts) != (k == parts - 1)) { printf("round %%d: block %%d of %%d\\n", round, k, parts); return 1; }
    }
    return 0;
}
""" % seed)


def test_whole_numbers_over_255_and_65280_are_rounded_as_a_division(tmp_path):
    run_host_program(tmp_path, """
template <int kDiv>
int check() {
    for (uint32_t v = 0; v <= (uint32_t)kDiv; ++v) {
        const volatile float n = (float)v, d = (float)kDiv;
        if (whole_over<kDiv>(v) != n / d) { printf("%u / %d\\n", v, kDiv); return 1; }
    }
    return 0;
}
int main() { return check<255>() | check<65280>(); }
""")

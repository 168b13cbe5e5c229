"""The rules by which the launchers of the LSTM cell choose a kernel (csrc/ktanh_order.h), compiled for the CPU: at the sizes
where a wrong choice was measured to cost time."""
import subprocess

import numpy as np

from paper_1909_07729_amd import build


def _run(tmp_path, body):
    src, exe = tmp_path / "forms.cpp", tmp_path / "forms"
    src.write_text('#include <cstdio>\n#include <vector>\n#include "ktanh_order.h"\nusing namespace ktanh_device;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout.strip() == "ok", (done.returncode, done.stdout, done.stderr[-2000:])


def test_when_the_backward_step_asks_for_what_is_no_gate_word(tmp_path):
    """At once on calls as long as one wavefront, late on calls that memory bounds; late loads are only built with the non-temporal hint, and
    loads at once only for whole pieces with plain ones."""
    _run(tmp_path, r"""
int main()
{
    for (unsigned long long H : {8, 40, 32, 64, 1000, 3072})
        for (bool lines : {false, true})
            for (unsigned long long n = 4; n < 1ull << 28; n += n / 37 + 1) {
                const bool is_short = cell_rows_are_short(H) && n >= 32768;
                const CellLoads want = is_short ? CELL_LOADS_IN_TURN
                                     : n <= 196608 ? CELL_LOADS_AT_ONCE
                                     : 60 * n > (lines ? 256ull : 128ull) << 20 ? CELL_LOADS_LATE : CELL_LOADS_IN_TURN;
                const CellBackward f = cell_backward_form(n, H, lines && !is_short);
                if (f.loads != want) return 1;
                if (f.loads == CELL_LOADS_AT_ONCE && (f.streamed || !f.whole)) return 2;
                if (f.loads == CELL_LOADS_LATE && !f.streamed) return 3;
            }
    std::puts("ok");
    return 0;
}
""")


def test_backward_step_of_rows_off_the_lines(tmp_path):
    """Stores that write through, in the plain order, cost up to 75 % more where neighbouring wavefronts share cache lines."""
    _run(tmp_path, r"""
static int is(unsigned long long B, unsigned long long H, unsigned long long pointers, bool streamed, bool whole)
{
    const CellBackward f = cell_backward_form(B * (H / 2), H, cell_rows_fill_lines(H, pointers));
    if (f.streamed == streamed && f.whole == whole) return 0;
    std::printf("B %llu H %llu pointers %llu: %d %d\n", B, H, pointers, f.streamed, f.whole);
    return 1;
}
int main()
{
    int bad = 0;
    for (unsigned long long H : {32, 64, 128, 1024, 3072})      // whole lines
        bad += is(1, H, 0, false, true) + is((47ull << 20) / (30 * H), H, 0, false, true) + is((52ull << 20) / (30 * H), H, 0, true, true) +
               is((400ull << 20) / (30 * H), H, 512, true, true);
    for (unsigned long long H : {72, 96, 1000, 1056, 3000})  // rows off the lines, and whole rows that start off them
        bad += is(1, H, 0, false, true) + is(1024, 1000, 0, false, true) + is((60ull << 20) / (30 * H), H, 0, false, false) +
               is((120ull << 20) / (30 * H), H, 0, true, false) + is((120ull << 20) / (30 * 1024), 1024, 4, true, false);
    for (unsigned long long H : {8, 16, 40, 56})            // short rows
        bad += is(1, H, 0, false, true) + is(((1 << 16) - 1) / H, H, 0, false, true) + is((1 << 16) / H + 1, H, 0, false, false) +
               is(100000, H, 0, false, false) + is(700000, H, 0, false, false);
    for (unsigned n : {1u, 63u, 32704u, 32705u, 32768u, 65537u, 1000003u}) {
        const unsigned tiles = (n + 63) / 64, runs = cell_run_tiles(n);
        std::vector<char> seen(tiles, 0);
        if (runs > tiles || tiles - runs >= kSpan) return 2;
        for (unsigned b = 0; b < tiles; ++b) {
            const unsigned t = tile_of_block_in_runs(b, runs, 0, 18);
            if (t >= tiles || seen[t]) return 3;
            seen[t] = 1;
        }
    }
    if (!bad) std::puts("ok");
    return bad;
}
""")


def test_single_step_of_rows_off_the_lines(tmp_path):
    """A large single step with the non-temporal hint in the plain order costs up to 9 % where neighbours share lines, and
    short rows need their lines in the cache."""
    _run(tmp_path, r"""
static int is(unsigned long long n, unsigned long long H, CellStep want)
{
    if (cell_step_form(n, H) == want) return 0;
    std::printf("%llu pairs H %llu: %d\n", n, H, cell_step_form(n, H));
    return 1;
}
int main()
{
    int bad = 0;
    for (unsigned long long H : {8, 32, 40, 64, 1000, 3000, 4096}) {
        const CellStep large = H == 8 || H == 40 ? STEP_SHORT_ROWS : STEP_STREAMED;
        bad += is(4, H, STEP_ONE_WAVE) + is(1 << 16, H, STEP_ONE_WAVE) + is((1 << 16) + 4, H, STEP_FOUR_WAVES) + is(1 << 19, H, STEP_FOUR_WAVES) +
               is((1 << 19) + 4, H, STEP_ONE_WAVE) + is(1 << 21, H, STEP_ONE_WAVE) + is((1 << 21) + 4, H, large) + is((1 << 28) - 4, H, large);
    }
    if (!bad) std::puts("ok");
    return bad;
}
""")


def test_two_stages_only_where_the_chip_is_full(tmp_path):
    """Two stages cover no latency by themselves: where the last round of blocks is mostly empty they cost up to 20 %."""
    _run(tmp_path, r"""
static int is(bool wide, unsigned T, unsigned n, bool shallow, unsigned H = 1024)
{
    if (shallow_ring(wide, T, n, H) == shallow) return 0;
    std::printf("wide %d T %u pairs %u H %u\n", wide, T, n, H);
    return 1;
}
int main()
{
    int bad = 0;
    for (unsigned T : {8, 12, 16, 32, 64}) {
        for (unsigned n : {4u, 262144u, 358400u, 527360u, 614400u, 716800u, 1049000u, 1100000u}) bad += is(false, T, n, false);
        for (unsigned n : {393216u, 435200u, 1u << 19, 870400u, 1u << 20, 1280000u, 1u << 21, (1u << 21) + 4, 4500000u, (1u << 28) - 4}) bad += is(false, T, n, true);
        for (unsigned n : {4u, 262144u, 460800u, 527360u, 614400u, 665600u}) bad += is(true, T, n, false);
        bad += is(true, T, 1u << 19, T < 16 || T >= 64) + is(true, T, 1u << 21, T >= 16) + is(true, T, 1u << 20, T >= 32);
    }
    bad += is(false, 0x7FFFFFFF, (1u << 28) - 4, true) + is(true, 0x7FFFFFFF, (1u << 28) - 4, true);   // no overflow
    for (unsigned H : {8, 16, 40, 56})                       // short rows
        for (unsigned n : {400000u, 460000u, 1u << 19, 870400u, 1u << 21}) bad += is(false, 16, n, false, H) + is(true, 32, n, false, H);
    for (unsigned H : {32, 72, 104, 136}) bad += is(false, 16, 460000, true, H) + is(false, 16, 1u << 19, false, H) + is(false, 16, 870400, true, H);
    for (unsigned H : {64, 96, 128, 160, 184, 1000}) bad += is(false, 16, 460000, true, H) + is(false, 16, 1u << 19, true, H);
    for (unsigned n : {527360u, 560000u, 1100000u}) bad += is(false, 16, n, false, 1000) + is(false, 16, n, false, 1024);
    for (unsigned n : {614400u, 720000u, 1150000u}) bad += is(false, 16, n, true, 1000) + is(false, 16, n, false, 1024);
    for (unsigned T : {2, 5, 7}) bad += is(false, T, (3u << 17) - 4, false) + is(false, T, 527360, true) + is(true, T, (1u << 19) - 4, false) + is(true, T, 527360, true);
    if (!bad) std::puts("ok");
    return bad;
}
""")


def test_ring_where_the_cells_do_not_fill_the_chip(tmp_path):
    """Four stages for few cells, three for more, none where the chip is full or rows off the lines cost more."""
    _run(tmp_path, r"""
static int is(unsigned T, unsigned n, unsigned long long H, unsigned stages, bool aligned = true)
{
    const unsigned got = ring_stages(T, n, H, aligned);
    if (got == stages) return 0;
    std::printf("T %u pairs %u H %llu aligned %d: %u\n", T, n, H, aligned, got);
    return 1;
}
int main()
{
    int bad = 0;
    for (unsigned T : {8u, 9u, 24u, 25u, 43u, 44u, 79u, 80u, 0x7FFFFFFFu}) {
        for (unsigned H : {64, 1024, 3072})
            bad += is(T, 32, H, 4) + is(T, 163840, H, 4) + is(T, 163844, H, 3) + is(T, (1u << 18) - 4, H, 3) + is(T, 1u << 18, H, 0);
        // many steps of whole rows that start off the lines: up to 5 % slower with the stages of the others
        for (unsigned H : {64, 2048})
            bad += is(T, 131072, H, 4, false) + is(T, 131076, H, T < 44 ? 4 : 0, false) + is(T, 163840, H, T < 44 ? 4 : 0, false) + is(T, 163844, H, T < 80 ? 3 : 0, false) + is(T, 1u << 18, H, 0, false);
        for (unsigned H : {8, 32, 40, 1000}) {
            const unsigned three = T <= 24 ? 3 : 0;
            bad += is(T, 4, H, 4) + is(T, 131072, H, 4) + is(T, 131076, H, three) + is(T, 196608, H, three) + is(T, 196612, H, 0) + is(T, (1u << 28) - 4, H, 0);
        }
    }
    for (unsigned H : {8, 64}) bad += is(7, 163840, H, 0) + is(1, 4, H, 0);
    for (unsigned H : {16, 64, 2048})
        for (unsigned T : {6u, 64u, 1u << 20}) bad += (full_ring_stages(T, (7u << 22) / T - 1, H) != 3) + (full_ring_stages(T, (7u << 22) / T + 1, H) != 2);
    // rows off the lines: up to 6 % slower with three stages
    for (unsigned H : {72, 200, 2000})
        for (unsigned T : {6u, 8u, 11u}) bad += (full_ring_stages(T, (3u << 18) - 4, H) != 3) + (full_ring_stages(T, 3u << 18, H) != 2) + (full_ring_stages(T, 1u << 21, H) != 2);
    bad += full_ring_stages(0x7FFFFFFF, (1u << 28) - 4, 2048) != 2;  // no overflow
    if (!bad) std::puts("ok");
    return bad;
}
""")


def test_chunks_of_time_where_they_gain(tmp_path):
    """A chunk of four whose last holds a single step costs up to 16 % near the end of the range of the others, and two steps never gain."""
    _run(tmp_path, r"""
static int last_in_chunks(unsigned T, unsigned n, unsigned steps)   // the largest size that chunks take, and how many steps it takes at a time
{
    int bad = 0;
    for (CellTable table : {CELL32, CELL64, CELL64_FOLDED})
        for (unsigned H : {8, 64, 1000}) {
            const CellForm f = cell_form(table, T, n, H);
            bad += f.kernel != CELL_CHUNKS || f.n != steps || cell_form(table, T, 4, H).kernel != CELL_CHUNKS || cell_form(table, T, n + 4, H).kernel == CELL_CHUNKS;
        }
    if (bad) std::printf("T %u pairs %u\n", T, n);
    return bad;
}
int main()
{
    int bad = last_in_chunks(3, 49152, 4) + last_in_chunks(4, 131072, 4) + last_in_chunks(5, 40960, 8) + last_in_chunks(6, 98304, 4) + last_in_chunks(8, 131072, 4);
    for (unsigned T : {9, 13, 17, 18, 19, 20, 33, 64, 65}) bad += last_in_chunks(T, 98304, 4);
    for (unsigned T : {10, 12, 14, 16}) bad += last_in_chunks(T, 114688, 4);
    for (unsigned T : {7, 11, 15}) bad += last_in_chunks(T, 131072, 4);
    for (unsigned n : {4u, 4096u, 49152u, (1u << 28) - 4}) bad += cell_form(CELL32, 2, n, 64).kernel != CELL_WRITTEN_OUT;
    bad += chunk_steps(64, 4096) != 64 || chunk_steps(64, 4100) != 32 || chunk_steps(64, 16384) != 32 || chunk_steps(64, 16388) != 16 || chunk_steps(64, 98304) != 4;
    // the byte offsets of a chunk's words, 16 per pair and step
    for (unsigned T : {3u, 4u, 7u, 16u, 17u, 64u, 90u, 0x7FFFFFFFu})
        for (unsigned n = 4; n < 1u << 28; n += n / 41 + 1) {
            const unsigned long long steps = chunk_steps(T, n);
            if (steps > 64 || 16 * steps * n > 1ull << 23) return 77;
        }
    if (!bad) std::puts("ok");
    return bad;
}
""")


def test_every_kernel_gets_only_steps_that_it_takes(tmp_path):
    """The ring fetches the steps of all its stages before it looks at their number, steps are written out for two to seven, and the lockstep and
    the multi-step kernel each are missing for one kind of table."""
    _run(tmp_path, r"""
int main()
{
    for (CellTable table : {CELL32, CELL64, CELL64_FOLDED})
        for (unsigned H : {8, 32, 40, 64, 96, 1000, 2048})
            for (unsigned T : {1u, 2u, 3u, 4u, 5u, 6u, 7u, 8u, 9u, 10u, 11u, 12u, 16u, 23u, 24u, 25u, 64u, 81u, 0x7FFFFFFFu})
                for (unsigned n = 4; n < 1u << 28; n += n / 397 + 1) {
                    const CellForm f = cell_form(table, T, n, H);
                    bool fine = false;
                    switch (f.kernel) {
                        case CELL_ONE_STEP: fine = T == 1; break;
                        case CELL_CHUNKS: fine = T >= 3 && f.n >= 4 && f.n <= 64 && (f.n & (f.n - 1)) == 0; break;
                        case CELL_RING_TOGETHER: fine = table != CELL64 && f.n == kTogetherStages && T >= f.n; break;
                        case CELL_RING: fine = (f.n == 3 || f.n == 4 || (f.n == 2 && table == CELL64_FOLDED)) && T >= f.n; break;
                        case CELL_WRITTEN_OUT: fine = T >= 2 && ((f.n == kDeepStages && T <= 7) || (f.n == kShallowStages && T <= 5)); break;
                        case CELL_MULTI_STEP: fine = table != CELL64_FOLDED && T >= 2 && (f.n == kDeepStages || f.n == kShallowStages); break;
                    }
                    if (!fine) {
                        std::printf("table %d T %u pairs %u H %u: kernel %d, %u\n", table, T, n, H, f.kernel, f.n);
                        return 1;
                    }
                }
    std::puts("ok");
    return 0;
}
""")


def test_large_blocks_where_their_last_round_is_nearly_full(tmp_path):
    """Blocks of 1024 pairs on 256 compute units: a last round that is mostly empty costs up to 30 %, most of all on short rows."""
    _run(tmp_path, r"""
static int from(unsigned T, unsigned H, unsigned first, unsigned last)   // blocks that are taken, next to ones that are not
{
    const int bad = rows_together(T, 1024 * (first - 1), H) || !rows_together(T, 1024 * (first - 1) + 4, H) || !rows_together(T, 1024 * last, H);
    if (bad) std::printf("T %u H %u blocks %u to %u\n", T, H, first, last);
    return bad;
}
int main()
{
    int bad = 0;
    for (unsigned H : {8, 32, 40, 48, 56, 72, 96, 2000}) {
        // up to 192 blocks of 1024 the others have three blocks of 256 on a compute unit
        for (unsigned T : {8, 9, 11, 12, 40, 96}) bad += from(T, H, 193, 256);
        for (unsigned T : {12, 16, 64}) bad += from(T, H, 256 + 208, 512) + from(T, H, 512 + (H < 40 ? 176 : H < 48 ? 128 : 120), 768) + from(T, H, 768 + 160, 1024);
        for (unsigned T : {16, 64}) {
            bad += H < 56 ? from(T, H, 1024 + (H < 40 ? 120 : 64), 1280) : !rows_together(T, 1024 * 1024 + 4, H);
            for (unsigned full : {5, 6, 7, 100}) bad += H < 40 && full < 7 ? from(T, H, 256 * full + (full == 5 ? 96 : 64), 256 * full + 256) : !rows_together(T, 1024 * 256 * full + 4, H);
        }
        bad += rows_together(15, 1024 * 1280, H) || rows_together(11, 1024 * 512, H) || rows_together(64, 1024 * 257, H);
    }
    for (unsigned H : {64, 2048}) {
        bad += from(8, H, 240, 256) + from(11, H, 240, 256) + from(24, H, 256 + 208, 512) + from(80, H, 256 + 208, 512) + rows_together(81, 1024 * 512, H) + from(16, H, 512 + 188, 768) + from(16, H, 768 + 240, 1024) + from(40, H, 1024 + 240, 1280);
        bad += rows_together(12, 1024 * 256, H) || rows_together(23, 1024 * 512, H) || rows_together(15, 1024 * 768, H) || rows_together(64, 1024 * 256, H);
    }
    for (unsigned H : {8, 64}) bad += rows_together(7, 1024 * 256, H) || rows_together(0, 1024 * 256, H) || rows_together(8, 0, H);
    bad += !rows_together(0x7FFFFFFF, (1u << 28) - 4, 8) || !rows_together(0x7FFFFFFF, (1u << 28) - 4, 64);   // no overflow
    if (!bad) std::puts("ok");
    return bad;
}
""")


COVERAGE = r"""
#include <map>
#include <set>
#include <string>
// The kernel of a call with what its code branches on: the length of a chunk and its blocks, the steps written out, the steps that are left behind a
// ring's steady loop.
static std::string key(CellTable table, unsigned T, unsigned n, unsigned long long H)
{
    const CellForm f = cell_form(table, T, n, H);
    unsigned left = T, detail = 0;
    if (f.kernel == CELL_RING_TOGETHER || f.kernel == CELL_RING || f.kernel == CELL_MULTI_STEP)
        if (T >= 2 * f.n) left = f.n + T % f.n;
    switch (f.kernel) {
        case CELL_ONE_STEP: detail = cell_step_form(n, H); break;
        case CELL_CHUNKS: detail = f.n == 32 ? T <= 32 && n <= 12288 : f.n == 4 ? chunk_words_at_once(T) : 0; break;
        case CELL_WRITTEN_OUT: detail = T; break;
        default: detail = left; break;
    }
    static const char *const names[] = {"one step, form", "chunks", "in lockstep, steps left", "ring, steps left", "written out", "multi-step, steps left"};
    return std::string(names[f.kernel]) + " " + std::to_string(f.n) + " " + std::to_string(detail);
}
int main()
{
    int bad = 0;
    for (CellTable table : {CELL32, CELL64, CELL64_FOLDED}) {
        std::set<std::string> reached, loose;
        for (unsigned i = 0; i < sizeof calls / sizeof *calls; ++i)
            if (calls[i][0] == table) {
                const std::string k = key(table, calls[i][1], calls[i][2] * (calls[i][3] / 2), calls[i][3]);
                reached.insert(k);
                if (calls[i][4]) loose.insert(k.substr(0, k.find_last_of(' ')));
            }
        std::map<std::string, std::string> all;
        for (unsigned T = 1; T < 70; ++T)
            for (unsigned H : {8, 32, 40, 64, 1000, 2048})
                for (unsigned n = 4; n < 1u << 23; n += (n / 61 + 4) & ~3u) {
                    char where[80];
                    std::snprintf(where, sizeof where, "T %u pairs %u H %u", T, n, H);
                    all.emplace(key(table, T, n, H), where);
                }
        for (const auto &k : all) {
            if (!reached.count(k.first)) { std::printf("table %d: no call of %s, as %s\n", table, k.first.c_str(), k.second.c_str()); ++bad; }
            // the kernels that carry a state of a table above 1 from step to step
            if (k.first[0] == 'o' || k.first[0] == 'c') continue;
            const std::string kernel = k.first.substr(0, k.first.find_last_of(' '));
            if (loose.insert(kernel).second) { std::printf("table %d: no call of %s with a table above 1, as %s\n", table, kernel.c_str(), k.second.c_str()); ++bad; }
        }
    }
    if (!bad) std::puts("ok");
    return bad != 0;
}
"""


def test_gpu_tests_reach_every_kernel_of_the_cell(tmp_path):
    """Every kernel that the launchers can take, with every remainder of its loop, is run by tests/test_gpu_variants.py: a line that moves does
    not take a kernel away from its tests unseen."""
    import test_gpu_variants as gpu
    calls = [(0, *s, 0) for s in gpu.CHUNKS + gpu.LINES + gpu.STEP + gpu.STEP_RUNS + gpu.ONE_NAN]
    calls += [(2, *s, 0) for s in gpu.WIDE + gpu.STEP + gpu.STEP_RUNS + gpu.ONE_NAN + [gpu.beyond_the_cache(T)[:3] for T in gpu.BEYOND]]
    calls += [(1, *s, 0) for s in gpu.NO_FOLD] + [(t, *s, 1) for s in gpu.LOOSE for t in (0, 1)] + [(2, *s, 1) for s in gpu.ABOVE_ONE]
    for T, B, _ in gpu.LOOSE:       # 4.0 is not taken to 1.0: the table does not fold
        E, _, b = gpu._any_valid_table(np.random.Generator(np.random.PCG64(T + B)), 64)[16]
        assert (E << 7) + b != 0x3F80
    _run(tmp_path, "static const unsigned calls[][5] = {%s};" % ", ".join("{%d, %d, %d, %d, %d}" % c for c in calls) + COVERAGE)

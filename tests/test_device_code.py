"""What the compiler made of the kernels, read from the gfx950 assembly of the shipped sources built
with the shipped flags: no packed Float32 arithmetic, no register spills to scratch memory, and the
table reads are the cross-lane instruction the design rests on."""
import os
import re
import subprocess

import pytest

from paper_1909_07729_amd import build

HIP_SOURCES = [s for s in build.SOURCES + build.PROBE_SOURCES if s.endswith(".hip")]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = {}
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    tmp = tmp_path_factory.mktemp("asm")
    procs = []
    for src in HIP_SOURCES:
        dst = str(tmp / (src + ".s"))
        cmd = [hipcc, *flags, "-S", "--cuda-device-only", "-I", os.path.join(build.ROOT, "include"),
               "-I", build.CSRC, os.path.join(build.CSRC, src), "-o", dst]
        procs.append((src, dst, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE)))
    for src, dst, p in procs:
        _, err = p.communicate(timeout=600)
        assert p.returncode == 0, err.decode()
        out[src] = open(dst).read()
    return out


def test_no_packed_float32_arithmetic(assembly):
    for src, text in assembly.items():
        hits = re.findall(r"v_pk_(?:add|mul|fma)_f32", text)
        assert not hits, f"{src}: {len(hits)} packed Float32 instructions"


def test_no_kernel_spills_registers(assembly):
    for src, text in assembly.items():
        sizes = [int(v) for v in re.findall(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", text)]
        assert sizes and all(v == 0 for v in sizes), f"{src}: private segment sizes {sizes}"
        assert "scratch_load" not in text and "scratch_store" not in text, src


def test_table_reads_are_cross_lane_and_stores_stream(assembly):
    # the streaming kernels' two kinds of store: past the last-level cache, and left in it
    for src, stores in (("ktanh_stream.hip", (r"global_store_dwordx4 .* sc0 sc1 nt", r"global_store_dwordx4 .* off sc1$")),
                        ("ktanh_backward.hip", (r"global_store_dwordx4 .* sc0 sc1 nt", r"global_store_dwordx4 .* off sc1$")),
                        ("ktanh_lstm.hip", (r"global_store_dword .* sc1$",))):
        text = assembly[src]
        assert "ds_bpermute_b32" in text, src
        assert "ds_read" not in text and "ds_write" not in text, f"{src}: the table must not live in LDS"
        for store in stores:
            assert re.search(store, text, flags=re.M), (src, store)
    assert re.search(r"global_load_dwordx4 .* nt", assembly["ktanh_stream.hip"])


def test_lstm_steady_loop_waits_for_its_own_gate_words_only(assembly):
    """With four register stages of four loads each, and the gate words of a step consumed one step
    early (its activations are formed under the previous step's wait), a step must wait for its four
    words with eight to eleven younger memory operations still in flight; a wait for everything
    (vmcnt(0)) inside the steady loop would serialise memory and arithmetic."""
    text = assembly["ktanh_lstm.hip"]
    loop = text[text.index("Inner Loop Header"):]
    loop = loop[:loop.index("s_endpgm")]
    for count in (11, 10, 9, 8):
        assert f"s_waitcnt vmcnt({count})" in loop, count
    steady = loop[:loop.index("ds_bpermute_b32")]          # the unrolled body up to the first out-of-line path
    assert "vmcnt(0)" not in steady


def _kernels(text, name):
    """{mangled name: code} of the kernels whose name contains `name`, code up to the first end of program."""
    parts = re.split(r"^(_Z\w+):", text, flags=re.M)
    return {n: body[:body.index("s_endpgm")] for n, body in zip(parts[1::2], parts[2::2]) if name in n and "s_endpgm" in body}


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("stages", [4, 2])
def test_every_ring_waits_for_its_own_gate_words_only(assembly, wide, stages):
    """The waits of the steady loop by the kernel's name: a step's four words arrive one by one, with the words of
    `stages` - 2 later steps still on their way.  Two stages thus leave nothing on its way while a step is computed."""
    kernels = _kernels(assembly["ktanh_lstm.hip"], f"lstm_cell_kernelILb{wide}ELb1ELi{stages}E")
    assert len(kernels) == 1
    code, = kernels.values()
    loop = code[code.index("Inner Loop Header"):]
    steady = loop[:loop.index("ds_bpermute_b32")]
    waits = [int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\)", steady)]
    assert waits == [4 * (stages - 2) + k for k in (3, 2, 1, 0)] * stages, waits
    assert steady.count("global_load_dword ") == 4 * stages and steady.count("global_store_dword ") == stages


def _steady_loop(code):
    """From the first loop's header to its last branch back."""
    label = re.search(r"^(\.LBB\d+_\d+):.*Inner Loop Header", code, flags=re.M)
    back = [m.end() for m in re.finditer(r"s_c?branch\w* " + re.escape(label.group(1)) + r"\b", code)]
    return code[label.start():back[-1]]


def test_ring_waits_for_its_own_gate_words_only(assembly):
    """A step asks for the words of the step STAGES ahead before it waits for its own, so that a wait leaves the words of STAGES - 1 steps on their way, and,
    except in lockstep, the stores in between; one step of the unrolled body asks behind its waits, which leave those of STAGES - 2.  No load or
    store has a branch around it."""
    found = _kernels(assembly["ktanh_lstm_ring.hip"], "lstm_ring_kernel")
    assert len(found) == 9
    for mangled, code in found.items():
        stages, threads = map(int, re.search(r"CellTableE\dELi(\d)ELi(\d+)E", mangled).groups())
        loop = _steady_loop(code)
        waits = [int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\)", loop)]
        fewer = [n for n in waits if n < 4 * (stages - 1)]
        assert len(waits) >= 3 * stages and len(fewer) <= 4 and min(waits) >= 4 * (stages - 2), (mangled, waits)
        if threads == 256 and stages > 2:   # a step's first word: all younger words and the stores of the steps between
            assert max(waits) > 4 * stages - 1, (mangled, waits)
        assert loop.count("global_load_dword ") == 4 * stages and loop.count("global_store_dword ") == stages, mangled
        assert loop.count("s_barrier") == (stages if threads == 1024 else 0), mangled
        assert "s_and_saveexec" not in loop, mangled


def test_late_loads_are_late(assembly):
    """dy behind x (2) or behind the slopes (3), and what the backward step asks for when the gates or K of the state are formed: the compiler would move them up."""
    for name, code in _kernels(assembly["ktanh_backward.hip"], "grad_stream_kernel").items():
        dy = int(re.search(r"DyLoadE(\d)E", name).group(1))
        ops = re.findall(r"global_load_dwordx4|s_waitcnt vmcnt\(0\)|ds_bpermute_b32", code)
        order = "".join({"g": "Q", "s": "w", "d": "."}[op[0]] for op in ops)
        body = order[:order.rindex("Q") + 1]        # up to the second load
        assert body.count("Q") == 2, (name, order)
        assert body == "QQ" if dy < 2 else body == "QwQ" if dy == 2 else re.fullmatch(r"Qw\.{4,}Q", body), (name, order)
    seen = set()
    for name, code in _kernels(assembly["ktanh_backward.hip"], "lstm_cell_backward_kernel").items():
        loads = int(re.search(r"CellLoadsE(\d)E", name).group(1))
        seen.add(loads)
        ops = re.findall(r"global_load_dword(?:x2)? |ds_bpermute_b32", code)
        order = "".join("." if op[0] == "d" else "D" if "x2" in op else "L" for op in ops)
        before, after = order.split(".", 1)[0], order.rstrip("DL")
        # the lane's table slot and the gate words first; c, dh and dc with them; or c with them and the rest behind the last table read; or c behind those of the gates
        with_gates, at_the_end = {0: (3, 0), 1: (1, 2), 2: (0, 2)}[loads]
        assert len(before) == 5 + with_gates and len(order) - len(after) == at_the_end, (name, order)
        assert order.count(".") == 10 and len(order) == 18, (name, order)
    assert seen == {0, 1, 2}


@pytest.mark.parametrize("src,kernels", [("ktanh_stream.hip", [f"13stream_kernelILb0ELi{op}ELb0E" for op in range(4)]),
                                         ("ktanh_backward.hip", [f"grad_stream_kernelItLi{grad}ELb0E" for grad in (2, 3)])])
def test_table_reads_of_a_vector_are_issued_together(assembly, src, kernels):
    """The eight table reads of a lane's eight BFloat16 values go out before the first of them is waited for: a small call has
    no other work to hide a latency per word."""
    for name in kernels:
        found = _kernels(assembly[src], name)
        assert found, name
        for mangled, code in found.items():
            order = "".join("." if "ds" in x else "|" for x in re.findall(r"s_waitcnt lgkmcnt\(\d+\)|ds_bpermute_b32", code))
            assert "." * 8 in order, (mangled, order)


def test_words_of_the_next_chunk_of_time_are_asked_for_where_they_gain(assembly):
    """In the loop of the chunk kernel: behind this chunk's table reads and before the walk, or, in short chunks of a long call, together with
    this chunk's words, whose waits then leave the stores of the chunk before in flight."""
    found = _kernels(assembly["ktanh_lstm_chunks.hip"], "lstm_chunk_kernel")
    assert len(found) == 21
    kinds = (("global_load_dword ", "L"), ("ds_bpermute_b32", "."), ("ds_write_b128", "W"), ("s_barrier", "B"), ("global_store_dword ", "S"))
    for mangled, code in found.items():
        at_once = re.search(r"CellTableE\dELi(\d+)ELi(\d+)ELb(\d)", mangled).groups() == ("64", "4", "1")
        ops = re.findall("|".join(k for k, _ in kinds), code)
        order = "".join(dict(kinds)[op] for op in ops)
        if at_once:
            assert "LLLL........W" in order, (mangled, order)
        else:
            assert "LLLL...." not in order[5:] and "........WLLLLB" in order, (mangled, order)


def test_gradients_form_all_slopes_first_only_where_that_gains(assembly):
    """Words in turn (0), all slopes first (1), dy behind x (2) or behind the slopes (3): Float32 gradients of a few MB are up to 6 % slower
    with all slopes first, GELU on aligned BFloat16 from 13 MiB moved on up to 4 %."""
    built = {}
    for name in _kernels(assembly["ktanh_backward.hip"], "grad_stream_kernel"):
        elem, grad, unaligned, near, dy = re.search(r"grad_stream_kernelI([tj])Li(\d)ELb\dELb(\d)ELb\dELb(\d)ELNS_6DyLoadE(\d)E", name).groups()
        built.setdefault((elem, int(grad), "near" if near == "1" else "off" if unaligned == "1" else "aligned"), set()).add(int(dy))
    for where in ("aligned", "off", "near"):
        late = set() if where == "near" else {3}
        assert built["j", 0, where] == built["j", 1, where] == {0} and built["j", 2, where] == built["j", 3, where] == {0} | late, where
        assert built["t", 0, where] == built["t", 1, where] == built["t", 2, where] == {1}, where
    assert built["t", 3, "aligned"] == {0, 1, 2} and built["t", 3, "off"] == {1, 2} and built["t", 3, "near"] == {1}


def test_wide_stores_written_as_statements_keep_their_data_registers(assembly):
    """A store of more than 64 bits reads its data registers for a few cycles after issue; the
    compiler inserts the wait for stores it emits itself but cannot see into a statement, so each such
    statement carries its own two idle slots."""
    seen = {True: 0, False: 0}
    for src, text in assembly.items():
        lines = text.splitlines()
        for i, line in enumerate(lines):
            if "global_store_dwordx4" in line and "sc1" in line:
                seen["sc0 sc1 nt" in line] += 1
                assert lines[i + 1].strip() == "s_nop 1", f"{src}: {line.strip()} is followed by {lines[i + 1].strip()}"
    assert seen[True] > 20 and seen[False] > 40, seen   # streamed past the last-level cache, left in it


def test_leading_scalar_arguments_are_preloaded(assembly):
    """Every streaming kernel gets the pointers and sizes it needs for its first load in registers."""
    for src in ("ktanh_stream.hip", "ktanh_backward.hip", "ktanh_probe.hip"):
        lengths = [int(v) for v in re.findall(r"\.amdhsa_user_sgpr_kernarg_preload_length\s+(\d+)", assembly[src])]
        assert lengths and min(lengths) >= 4, (src, sorted(set(lengths)))


def test_the_yardstick_of_the_cell_takes_the_multi_step_kernel_with_either_table(tmp_path):
    """Without arithmetic there is the multi-step kernel alone: the ring of ktanh_lstm_ring.hip would compute, and reads its
    stages' steps whether a call has them or not."""
    src, obj = tmp_path / "yardstick.hip", tmp_path / "yardstick.o"
    src.write_text("""#include "ktanh_lstm_impl.h"
using namespace ktanh_device;
template ktanh_status_t ktanh_device::launch_cell<false, false, ktanh_lut_t>(const uint16_t *, const float *, float *, uint16_t *, size_t, size_t, size_t, const ktanh_lut_t *, ktanh_stream_t);
template ktanh_status_t ktanh_device::launch_cell<true, false, ktanh_lut64_t>(const uint16_t *, const float *, float *, uint16_t *, size_t, size_t, size_t, const ktanh_lut64_t *, ktanh_stream_t);
""")
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-host-only", "-c", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, str(src), "-o", str(obj)], check=True)
    names = subprocess.run(["nm", "-C", str(obj)], capture_output=True, text=True, check=True).stdout
    assert "lstm_cell_kernel<true, false, 4>" in names and "lstm_cell_kernel<false, false, 2>" in names
    assert not re.findall(r"launch_cell_(?:ring|chunks)|lstm_(?:ring|chunk|short|step)_kernel", names)

"""Properties of the compiled kernels that their sources rely on and no run can show: read from the assembly that the
compiler writes for this library's own files (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2512_06547_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    done = {}

    def of(name):
        if name not in done:
            out = str(tmp_path_factory.mktemp("asm") / (name + ".s"))
            subprocess.check_call([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, name),
                                   "-o", out], stderr=subprocess.DEVNULL)
            with open(out) as f:
                done[name] = f.read()
        return done[name]

    return of


def kernels(text, name):
    """{mangled name: body} of the kernels whose name holds `name`."""
    found = {m.group(1): m.group(2) for m in
             re.finditer(r"^(_ZN4a3po\w*" + name + r"\w*):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S | re.M)}
    assert found, f"no kernel {name}"
    return found


def memory_events(body):
    """The vector memory operations, waits on them and barriers of a kernel, in program order."""
    events = []
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        op = line.split(" ")[0] if line else ""
        if re.match(r"(global|buffer|flat|scratch)_(load|store)", op):
            events.append("direct" if line.endswith(" lds") else op)
        elif op == "s_barrier":
            events.append("barrier")
        elif op == "s_waitcnt" and "vmcnt" in line:
            events.append(int(re.search(r"vmcnt\((\d+)\)", line).group(1)))
    return events


@pytest.mark.parametrize("blocks", [4, 8, 12, 16])
def test_few_token_kernel_issues_loads_in_the_counted_order(assembly, blocks):
    """lmhead_few_tokens_kernel waits for its hidden rows by a number of operations that may still be in flight, which
    holds for one order of issue: weight and hidden rows of a chunk in turn before the loop (no hidden rows for the
    fourth chunk), then per chunk the hidden rows three chunks ahead and the weight four ahead.  No wait in the loop may
    ask for more than that number either: it would drain the weight's loads."""
    body, = kernels(assembly("a3po_lmhead.hip"), f"lmhead_few_tokens_kernelILi{blocks}E").values()
    events, direct, load = memory_events(body), ["direct"] * (blocks // 4), ["global_load_dwordx4"] * 4
    wait = [12 + 2 * (blocks // 4), "barrier"]
    steady = (load + direct) * 3 + load + (wait + direct + load) * 4
    first = events.index("barrier")
    assert events[:len(steady)] == steady, events[:max(first + 1, len(steady))]


@pytest.mark.parametrize("product", ["Lse", "LseStore", "SplitRows", "SplitPanels", "PanelsBf16", "PanelsF32"])
def test_contraction_epilogue_leaves_the_ring_in_flight(assembly, product):
    """gemm_kernel writes a tile out while the direct loads of the next one arrive: between the waits that are counted by
    hand (12 operations in flight before the loop, 8 per stage) and the one at the kernel's end it waits for no vector
    memory operation - which a spilled register, or an access to the staging tiles or column partials that the compiler holds
    for one to the ring, would bring.  (The products with the log-sum-exp have a second form, whose loop is two stages long.)"""
    number = {"Lse": 0, "LseStore": 1, "SplitRows": 2, "SplitPanels": 3, "PanelsBf16": 4, "PanelsF32": 5}[product]
    found = kernels(assembly("a3po_gemm.hip"), f"gemm_kernelILi{number}E")
    assert len(found) == (2 if number < 2 else 1)
    for name, body in found.items():
        events = memory_events(body)
        assert not [e for e in events if str(e).startswith("scratch")]
        assert [e for e in events if isinstance(e, int)] == [12] + [8] * (4 if "Lb1E" in name else 2) + [0]


@pytest.mark.parametrize("number", range(6))
def test_contraction_loop_computes_addresses_in_scalar_registers(assembly, number):
    """Every direct load of gemm_kernel's K loop takes a scalar base and a 32-bit lane offset; 64-bit vector additions
    between the matrix instructions cost the products of panel operands 2 to 5 %."""
    (name, body), = [(n, b) for n, b in kernels(assembly("a3po_gemm.hip"), f"gemm_kernelILi{number}ELb1E").items()]
    loop = max(re.split(r"\n\.?LBB\w+:", body), key=lambda block: block.count("v_mfma"))
    assert loop.count("v_mfma") == 4 * 32 and loop.count("global_load_lds_dwordx4") == 4 * 4
    assert not re.findall(r"v_lshl_add_u64|v_mad_[ui]64|v_add_co|v_readfirstlane", loop)


def vector_spills(text):
    """[(kernel, vector registers it spills)] of a file's assembly."""
    found = re.findall(r"\.name:\s+(_ZN4a3po\w+)\n(?:(?!\.name:).)*?\.vgpr_spill_count:\s+(\d+)", text, re.S)
    return [(name, int(n)) for name, n in found]


def test_row_kernels_keep_their_rows_in_registers(assembly):
    """The register-resident rows are only that if the compiler does not spill them: a handful of addresses may go to
    scratch memory (15 registers at most), rows may not."""
    spills = vector_spills(assembly("a3po_rows.hip"))
    assert len(spills) > 100
    assert not [(name, n) for name, n in spills if n > 15]


def test_short_batch_kernels_spill_nothing(assembly):
    """They hold a few vectors and one token's terms: nothing in them needs scratch memory, with or without the entropy."""
    spills = vector_spills(assembly("a3po_few.hip"))
    assert len(spills) == 16
    assert not [(name, n) for name, n in spills if n > 0]


@pytest.mark.parametrize("blocks", [12, 16])
def test_few_token_kernel_with_one_row_block_waits_for_its_own_count(assembly, blocks):
    """The last round's loop without second row blocks has two weight loads per chunk, and its waits allow for no more: what
    may be in flight behind a chunk's hidden rows is three chunks' weight and two chunks' hidden rows."""
    body, = kernels(assembly("a3po_lmhead.hip"), f"lmhead_few_tokens_kernelILi{blocks}E").values()
    events, direct, load = memory_events(body), ["direct"] * (blocks // 4), ["global_load_dwordx4"]
    wait = [6 + 2 * (blocks // 4), "barrier"]
    first = events.index(wait[0])
    assert events[first:first + 4 * (2 + len(direct) + 2)] == (wait + direct + load * 2) * 4, events[first:]

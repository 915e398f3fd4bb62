"""What the compiler leaves to the source, looked up in the library that was built from it (AMD machine code): no device needed."""
import os
import re
import subprocess

import pytest

import paper_2309_13541_amd as a2a

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    at = tmp_path_factory.mktemp("code")
    lib = at / "lib.so"
    lib.symlink_to(a2a.library_path())
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, timeout=120)
    objects = sorted(str(p) for p in at.iterdir() if p.name.endswith("gfx950"))
    assert len(objects) == 6  # one per translation unit
    return objects


def registers(operand):
    m = re.fullmatch(r"([vs])(\d+|\[(\d+):(\d+)\])", operand)
    if not m:
        return {operand} & {"m0", "vcc"}
    first, last = (m[2], m[2]) if m[3] is None else (m[3], m[4])
    return {m[1] + str(i) for i in range(int(first), int(last) + 1)}


def loads_to_lds_too_early(lines):
    """Loads to LDS, and those with too few wait states behind a scalar write of M0 (1) or a vector write of their scalar
    registers (5).  In the order of the text: the library's loads to LDS stand in one block with what they wait for."""
    found, early, before = 0, [], []
    for line in lines:
        text = line.split("//")[0].strip()
        op, _, rest = text.partition(" ")
        operands = [x.strip().split(" ")[0] for x in rest.split(",")]
        if "_lds_dword" in op:
            found += 1
            scalars = {r for x in operands for r in registers(x) if r[0] == "s"}
            states = 0
            for was, writes, waits in reversed(before):
                if (states < 1 and was[:2] == "s_" and "m0" in writes) or (states < 5 and was[:2] == "v_" and writes & scalars):
                    early.append(f"{was} {sorted(writes)}, {states} wait states: {text}")
                states += waits
        waits = int(operands[0], 0) + 1 if op == "s_nop" else 1
        before = before[-5:] + [(op, registers(operands[0]), waits)]
    return found, early


def test_the_check_itself():
    write, load = "s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]"
    for lines, bad in (([write, load], 1), ([write, "s_nop 0", load], 0), ([write, "v_add_u32_e32 v2, v3, v4", load], 0),
                       (["v_readlane_b32 s3, v9, 1", write, "s_nop 2", load], 1),
                       (["v_readlane_b32 s3, v9, 1", write, "s_nop 3", load], 0), (["v_readlane_b32 s5, v9, 1", "s_nop 0", load], 0)):
        assert loads_to_lds_too_early(lines)[0] == 1 and len(loads_to_lds_too_early(lines)[1]) == bad, lines


def test_loads_to_lds_wait_for_their_registers(code_objects):
    """The write of M0 and the load are one piece of assembly, in which the compiler keeps no wait states."""
    found = 0
    for path in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", path], check=True, stdout=subprocess.PIPE,
                              text=True, timeout=120).stdout
        n, early = loads_to_lds_too_early(text.splitlines())
        assert not early, early[:5]
        found += n
    assert found > 0


CSRC = os.path.join(os.path.dirname(a2a.library_path()), "csrc")


def by_address():
    """Kernels that use LDS by its byte address, by themselves or through what they call (by name: rather more than fewer)."""
    head = re.compile(r"__(global|device)__\b[^;({}]*?(\w+)\s*\(")
    text, kernels = {}, set()  # of a function: from its head to the next one's
    for name in sorted(os.listdir(CSRC)):
        if name.endswith(".h"):
            with open(os.path.join(CSRC, name)) as f:
                source = re.sub(r"//.*|__launch_bounds__\(\w+\)", "", f.read())
            heads = list(head.finditer(source))
            for m, end in zip(heads, [m.start() for m in heads[1:]] + [len(source)]):
                text[m[2]] = text.get(m[2], "") + source[m.end():end]
                if m[1] == "global":
                    kernels.add(m[2])
    users = {"lds_get", "lds_put"}
    while True:
        calls = re.compile(rf"\b(?:{'|'.join(sorted(users))})\s*[<(]")
        more = {f for f in text if f not in users and calls.search(text[f])}
        if not more:
            return users & kernels
        users |= more


def test_lds_by_address_starts_at_zero(code_objects):
    """Such a kernel has no LDS but its dynamic array: no __shared__ array of its own or of what it calls."""
    names = by_address()
    assert names >= {"k_small_loads", "k_small_sigma", "k_small_dist", "k_small_levels", "k_flow_sources", "k_flow_links", "k_flow_sssp"}
    assert not names & {"k_wide_dist", "k_small_sssp", "k_small_reduce"}  # these have some
    sizes = {}
    for path in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, stdout=subprocess.PIPE, text=True,
                               timeout=120).stdout
        for size, length, rest in re.findall(r"\.group_segment_fixed_size: (\d+)(?:.*\n)+?.*\.name: +_ZN7a2a_devL?(\d+)(\w+)", notes):
            sizes.setdefault(rest[:int(length)], set()).add(int(size))
    assert names <= set(sizes) and 0 not in sizes["k_wide_dist"]
    assert {k: sizes[k] for k in names if sizes[k] != {0}} == {}


def test_registers_of_a_thread_per_node(code_objects):
    """Link loads with a thread per node, a source at a time, keep all of a thread's nodes in registers: only 10 links of two
    nodes with demands do not fit."""
    scratch = {}
    for path in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, stdout=subprocess.PIPE, text=True,
                               timeout=120).stdout
        for words, nodes, sources, demand, size in re.findall(
                r"\.name: +_ZN7a2a_dev12k_node_loadsILi(\d)ELi(\d)ELi(\d)ELb(\d)E\w*\n.*\.private_segment_fixed_size: (\d+)", notes):
            scratch[int(words), int(nodes), int(sources), int(demand)] = int(size)
    alone = {k: v for k, v in scratch.items() if k[2] == 1}
    assert len(alone) == 18  # 2 to 5 words: a node or two a thread, 8 words: one
    assert alone.pop((5, 2, 1, 1)) <= 32
    assert {k: v for k, v in alone.items() if v} == {}


def test_words_in_memory_between_the_sweeps_of_a_strip_source():
    """lds_barrier() waits for LDS only.  Where k_strip_sources begins to read the records that other threads have stored, a
    barrier for memory stands before it, and a record is no place outside the link table whatever it holds."""
    with open(os.path.join(CSRC, "a2a_flow_kernels.h")) as f:
        source = re.sub(r"//.*", "", f.read())
    kernel = re.split(r"k_strip_sources\(FlowView fv\) \{", source)[1].split("__global__")[0]
    stored = kernel.index("lds_at(record, 4u * (uint32_t)(a.base + tt)) =")
    read = kernel.index("= lds_at(record,", stored)
    assert "__syncthreads();" in kernel[stored:read]
    # (a thread's own records, and nodes of the queue, are no other thread's)
    rows = re.findall(r"\.load\(fv\.out, (.*)\);", kernel)
    assert len(rows) >= 6 and all(row.startswith("min(") for row in rows if "r[" in row), rows

"""Orders between wavefronts that no run can be relied on to show, checked in the machine code of the built library.

A barrier waits for the wavefront's LDS operations, not for its stores to memory, and a fence waits for the stores of the
wavefront that executes it: what one thread publishes for its workgroup needs a wait for stores in front of the barrier."""
import os
import re
import subprocess

import pytest

import paper_2502_20969_amd.build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MERGES = ["_ZN3ivf12merge_kernelILi512EEEvNS_9MergeArgsE", "_ZN3ivf12merge_kernelILi1024EEEvNS_9MergeArgsE",
          "_ZN3ivf17merge_wide_kernelENS_9MergeArgsE"]
REDO = "_ZN3ivf17exact_redo_kernelENS_8RedoArgsE"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """symbol -> its instructions: [(place in the kernel, text, place a branch leads to)]"""
    at = tmp_path_factory.mktemp("code")
    os.symlink(B.LIB, at / "libivf.so")
    subprocess.run([OBJDUMP, "--offloading", "libivf.so"], cwd=at, check=True, capture_output=True)
    found = {}
    for f in sorted(p for p in os.listdir(at) if "gfx950" in p):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(MERGES + [REDO]), f], cwd=at,
                           check=True, capture_output=True, text=True)
        for line in r.stdout.splitlines():
            head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if head:
                body, first = found.setdefault(head.group(1), []), int(line.split()[0], 16)
            elif line.startswith("\t"):
                m = re.match(r"\t(.*?)\s*// ([0-9A-F]+):[^<]*(?:<\S+?(?:\+0x([0-9a-f]+))?>)?", line)
                if m:
                    body.append((int(m.group(2), 16) - first, m.group(1), int(m.group(3) or "0", 16)))
    return found


def _waits_for_stores(body, at):
    """Whether the barrier in front of instruction `at` stands behind a wait for stores, with no store or branch in between."""
    while body[at][1] != "s_barrier":
        at -= 1
    while at > 0:
        at -= 1
        if "vmcnt(0)" in body[at][1]:
            return True
        if re.match(r"global_(store|atomic)|flat_|buffer_|s_cbranch|s_branch", body[at][1]):
            return False
    return False


@pytest.mark.parametrize("kernel", MERGES)
def test_completion_word_is_stored_behind_everyones_results(code, kernel):
    body = code[kernel]
    word = [i for i, (_, t, _) in enumerate(body) if t.startswith("global_store_dwordx2") and t.endswith("sc0 sc1")]
    assert len(word) == 1
    assert _waits_for_stores(body, word[0])


def test_ticket_of_the_exact_pass_is_drawn_behind_everyones_lists(code):
    """The workgroup that draws the last ticket reads the lists of the others, which may have run beside another L2."""
    body = code[REDO]
    ticket = [i for i, (_, t, _) in enumerate(body) if t.startswith("global_atomic_add")]
    assert len(ticket) == 1
    assert _waits_for_stores(body, ticket[0])


@pytest.mark.parametrize("kernel", MERGES)
def test_pool_size_is_reset_behind_everyones_read(code, kernel):
    """Every wavefront branches on the number of pooled candidates, a word of LDS that later steps start again from zero:
    on no path from a read of it to a store that resets it may a barrier be missing."""
    body = code[kernel]
    place = {a: i for i, (a, _, _) in enumerate(body)}
    counters = {re.search(r"offset:\d+", t).group() for _, t, _ in body if t.startswith("ds_add_rtn_u32")}
    assert counters                                              # wavefronts take their places in the pool
    reads, resets = [], {}
    for i, (_, t, _) in enumerate(body):
        word = re.search(r"offset:\d+", t)
        if word and word.group() in counters and t.startswith("ds_read_b32"):
            reads.append((i, word.group()))
        if word and word.group() in counters and t.startswith("ds_write"):
            resets[i] = word.group()
    assert reads and resets
    for read, word in reads:
        seen, todo = set(), [read + 1]
        while todo:
            i = todo.pop()
            if i in seen or body[i][1] in ("s_barrier", "s_endpgm"):
                continue
            seen.add(i)
            assert resets.get(i) != word, f"instructions {read} .. {i}"
            if body[i][1].startswith(("s_branch", "s_cbranch")):
                todo.append(place[body[i][2]])
            if not body[i][1].startswith("s_branch"):
                todo.append(i + 1)

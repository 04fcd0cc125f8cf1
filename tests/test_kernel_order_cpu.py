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


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """symbol -> its instructions: [(address, text, branch target from the start of the kernel)]"""
    at = tmp_path_factory.mktemp("code")
    os.symlink(B.LIB, at / "libivf.so")
    subprocess.run([OBJDUMP, "--offloading", "libivf.so"], cwd=at, check=True, capture_output=True)
    found = {}
    for f in sorted(p for p in os.listdir(at) if "gfx950" in p):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(MERGES), f], cwd=at,
                           check=True, capture_output=True, text=True)
        for line in r.stdout.splitlines():
            head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if head:
                body = found.setdefault(head.group(1), [])
            elif line.startswith("\t"):
                m = re.match(r"\t(.*?)\s*// ([0-9A-F]+):[^<]*(?:<\S+?(?:\+0x([0-9a-f]+))?>)?", line)
                if m:
                    body.append((int(m.group(2), 16), m.group(1), int(m.group(3) or "0", 16)))
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

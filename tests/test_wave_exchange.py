"""Data passed between lanes of a wave, checked in the LLVM IR of the kernels.

Where lanes read from LDS what other lanes of their wave wrote, without a
workgroup barrier, the compiled code must keep the accesses in order: it may
otherwise hand a lane the value that the lane itself wrote.  The order is a wave
barrier between fences.

Where one lane alone runs, no register of another lane may be read: if that
value is spilled, only the running lane's part is loaded back for the read."""
import re
import subprocess

import pytest

from paper_2609_35629_amd.build import CFLAGS, CSRC, hipcc


def _kernels(src, name, tmp_path):
    ir = str(tmp_path / "k.ll")
    r = subprocess.run([hipcc(), *CFLAGS, "--offload-device-only", "-emit-llvm", "-S", f"{CSRC}/{src}", "-o", ir],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(ir) as f:
        found = re.findall(r"^define[^\n]*" + name + r".*?^}", f.read(), re.M | re.S)
    assert found
    return found


def _ordered(text):
    """Whether the text holds release fence, wave barrier, acquire fence."""
    return re.search(r'syncscope\("wavefront"\) release.*?wave\.barrier.*?syncscope\("wavefront"\) acquire', text, re.S)


def test_team_marks_of_the_routing_kl(tmp_path):
    # lane's own mark stored, other lanes' marks by atomic maximum, then read
    for body in _kernels("diag_kernels.hip", "k_kl_rows", tmp_path):
        marks = [m.start() for m in re.finditer(r"atomicrmw max ptr addrspace\(3\)", body)]
        assert len(marks) == 1
        store = body.rfind("store i32", 0, marks[0])
        load = re.compile(r"load i32, ptr addrspace\(3\)").search(body, marks[0]).start()
        assert _ordered(body[store:marks[0]])
        assert _ordered(body[marks[0]:load])


def test_member_offsets_of_the_parent_lists(tmp_path):
    # each group of 64 tokens reads its labels' offsets, then one lane per
    # label moves the label's offset on for the next group
    for body in _kernels("kmeans_kernels.hip", "k_parent_lists", tmp_path):
        place = body[body.rfind("s.barrier"):]
        acc = [(m.start(), m.group(1)) for m in re.finditer(r"\b(load|store) i32[^\n]*ptr addrspace\(3\)", place)]
        assert len(acc) >= 4
        for (a, x), (b, y) in zip(acc, acc[1:]):
            assert x == y or _ordered(place[a:b]), place[a:b]


@pytest.mark.parametrize("src,name", [("build_kernels.hip", "k_build"), ("kmeans_kernels.hip", "k_k"),
                                      ("diag_kernels.hip", "k_")])
def test_one_lane_reads_no_other_lane(src, name, tmp_path):
    for body in _kernels(src, name, tmp_path):
        lane = set(re.findall(r"^  (%\S+) = and i32 %\S+, 63$", body, re.M))
        first = {m.group(1) for m in re.finditer(r"^  (%\S+) = icmp eq i32 (%\S+), 0$", body, re.M) if m.group(2) in lane}
        blocks = dict(re.findall(r"^(\d+|[\w.]+):.*?\n(.*?)(?=^\S|\Z)", body, re.M | re.S))
        for m in re.finditer(r"br i1 (%\S+), label %(\S+), label %", body):
            if m.group(1) in first:
                assert not re.search(r"amdgcn\.(readlane|update\.dpp|ds\.bpermute)", blocks[m.group(2).rstrip(",")]), m.group(0)

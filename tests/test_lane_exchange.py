"""Rows of merged buckets are looked up in other lanes' registers (buffer_row in csrc/ffn_plan.h).  That is sound only
where every lane is active: a register that the compiler refills or copies inside a branch holds nothing for the lanes
that do not take it.  Checked on the AMD assembly that hipcc makes of the kernels; no GPU is needed or touched."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_06643_amd import build

OPENS = re.compile(r"s_(?:and|andn2|or)_saveexec_b64 (\S+),")
CLOSES = re.compile(r"s_or_b64 exec, exec, (\S+)")


def masked_lane_reads(asm):
    """(kernel, lane reads, those of them that some path reaches with lanes masked off) of every kernel."""
    for kernel, body in re.findall(r"^(_Z\w+):.*?$(.*?)^\.Lfunc_end", asm, re.M | re.S):
        blocks, name = {"entry": []}, "entry"
        order = ["entry"]
        for line in body.splitlines():
            m = re.match(r"(\.LBB\w+):", line)
            if m:
                name = m.group(1)
                blocks[name] = []
                order.append(name)
            elif re.match(r"\s+[sv]_", line):
                blocks[name].append(line.split(";")[0].strip())
        reads, masked, seen, todo = set(), set(), set(), [("entry", 0, ())]
        while todo:                                  # the masks that are open when a block is entered: every path
            block, i, opened = todo.pop()
            if (block, i, opened) in seen:
                continue
            seen.add((block, i, opened))
            code = blocks[block]
            while i < len(code):
                op = code[i]
                m = OPENS.match(op)
                if m and m.group(1) not in opened:
                    opened += (m.group(1),)
                m = CLOSES.match(op)
                if m and m.group(1) in opened:
                    opened = opened[:opened.index(m.group(1))]
                if op.startswith("v_readlane"):
                    reads.add((block, i))
                    if opened:
                        masked.add((block, i))
                i += 1
                m = re.match(r"s_c?branch\S* (\.LBB\w+)", op)
                if m:
                    todo.append((m.group(1), 0, opened))
                if op.startswith(("s_branch", "s_endpgm")):
                    break
            else:
                if order.index(block) + 1 < len(order):
                    todo.append((order[order.index(block) + 1], 0, opened))
        yield kernel, len(reads), len(masked)


@pytest.mark.parametrize("source", ["ffn_bf16", "ffn_skinny", "ffn_f32"])
def test_lane_reads_happen_with_all_lanes_active(tmp_path, source):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    out = tmp_path / "k.s"
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source + ".hip"), "-o", str(out)], check=True,
                   capture_output=True, timeout=300)
    found = [k for k in masked_lane_reads(out.read_text()) if k[1]]
    assert found, "no kernel reads lanes: the check looks for the wrong instruction"
    assert [k for k in found if k[2]] == []

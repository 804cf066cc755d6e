"""The head_dim 64 attention kernel refills an LDS buffer right behind a barrier, so no LDS read
may be outstanding at any of its barriers: the barrier alone does not wait for them, and a load
of another wave could then overwrite what they read.  Checked on the kernel's assembly, over
every path of its control flow."""
import os
import re
import subprocess

import pytest

from paper_2606_00487_amd import build as B

BRANCH = re.compile(r"s_c?branch\w*\s+(\S+)")


def outstanding_reads(lines):
    """Lines of the s_barriers that LDS reads may still be in flight at, over all paths.

    A state holds, oldest first, whether each LDS operation that may be in flight is a read:
    LDS operations finish in order, and lgkmcnt(n) leaves at most the newest n of them."""
    at = {m.group(1): k for k, s in enumerate(lines) if (m := re.match(r"(\S+):", s))}
    join = lambda a, b: tuple(x | y for x, y in zip(*((0,) * (64 - len(s)) + s for s in (a, b))))
    seen, todo, found = {}, [(0, ())], set()
    while todo:
        k, st = todo.pop()
        while k < len(lines):
            s = lines[k].split("//")[0].split(";")[0].strip()
            if s.endswith(":"):
                new = join(st, seen.get(k, ()))
                if seen.get(k) == new:
                    break
                seen[k] = st = new
            elif s.startswith("ds_"):
                st = (st + (int(s.startswith(("ds_read", "ds_load"))),))[-64:]
            elif s.startswith("s_waitcnt"):
                if m := re.search(r"lgkmcnt\((\d+)\)", s):
                    st = st[len(st) - min(len(st), int(m.group(1))):]
            elif s.startswith("s_barrier"):
                if any(st):
                    found.add(k)
            elif m := BRANCH.match(s):
                todo.append((at[m.group(1)], st))
                if s.startswith("s_branch"):
                    break
            elif s.startswith("s_endpgm"):
                break
            k += 1
    return sorted(found)


@pytest.mark.parametrize("wait,found", [
    ("s_waitcnt lgkmcnt(0)", []), ("s_waitcnt lgkmcnt(1)", [5]), ("s_waitcnt vmcnt(0)", [5])])
def test_the_check_itself(wait, found):
    """A read that is waited for on one path into the loop and, with less than a full wait in
    the loop's body, not on the other."""
    assert outstanding_reads(["f:", "s_waitcnt lgkmcnt(0)", "L:", "ds_read_b128 v[0:3], v4", wait,
                              "s_barrier", "s_cbranch_scc1 L", "s_endpgm"]) == found


def test_no_read_in_flight_at_a_barrier_of_the_head_dim_64_kernel():
    cmd = [B.hipcc(), *B.COMMON, *B.PER_FILE["attn.hip"], "-x", "hip", "--cuda-device-only", "-S",
           os.path.join(B.CSRC, "attn.hip"), "-o", "-"]
    asm = subprocess.run(cmd, capture_output=True, text=True, check=True).stdout.split("\n")
    begin = [k for k, s in enumerate(asm) if re.match(r"_ZN\w*attn_bf16_w4_kernel\w*:", s)]
    assert len(begin) == 1
    body = asm[begin[0]:next(k for k in range(begin[0], len(asm)) if ".end_amdhsa_kernel" in asm[k]
                             or asm[k].startswith(".Lfunc_end"))]
    assert sum("s_barrier" in s for s in body) >= 8 and sum("ds_read" in s for s in body) >= 64
    bad = outstanding_reads(body)
    assert not bad, [body[k - 3:k + 1] for k in bad]

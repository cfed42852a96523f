"""What the kernels' sources must not contain."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_02337_amd", "csrc")


def test_no_load_in_assembly_outlives_its_statement():
    """A load that inline assembly issues and does not wait for lands in a register that the compiler takes to hold its
    result already: it may have put something else there by then, an address for instance.  Every asm statement that
    loads into registers (from memory or LDS) waits for all of it before it ends."""
    loads = re.compile(r"\b(global|flat|buffer|scratch)_load_\w*|\bds_read\w*|\bs_load_\w*")
    found = 0
    for f in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = re.sub(r"//[^\n]*", "", open(f).read())
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(\s*((?:\"(?:\\.|[^\"])*\"\s*)+)", text):
            body = "".join(re.findall(r"\"((?:\\.|[^\"])*)\"", m.group(1)))
            ops = [x for x in (y.replace("\\t", " ").strip() for y in body.split("\\n")) if x]
            kinds = [loads.search(o) for o in ops]
            if not any(kinds):
                continue
            found += 1
            memory = any(k and not k.group(0).startswith(("ds_", "s_")) for k in kinds)
            last = ops[-1]
            assert last.startswith("s_waitcnt") and ("vmcnt(0)" if memory else "lgkmcnt(0)") in last, (os.path.basename(f), body)
    assert found >= 4   # the LDS reads of attn_mfma.h

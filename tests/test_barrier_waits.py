"""Every workgroup barrier of the compiled kernels is reached with the
wavefront's LDS writes complete: on no path from an LDS write to an s_barrier
is the s_waitcnt missing.  (A loop whose barrier stood at its head had its wait
before the loop only; a tree's block maxima were then now and then wrong.)"""
import glob
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_1309_3458_amd import build_lib as B

LIMIT = 64  # LDS operations counted after a write


def functions(text):
    """{name: [(label, [instruction])]}, in order"""
    out, blocks = {}, None
    for line in text.splitlines():
        line = line.split(";")[0].rstrip()
        if re.match(r"[A-Za-z_]\w*:", line):
            blocks = out.setdefault(line[:-1], [("", [])])
        elif blocks is None:
            continue
        elif re.match(r"\.LBB\w+:", line):
            blocks.append((line[:-1], []))
        elif line.strip() and not line.strip().startswith("."):
            blocks[-1][1].append(line.split())
    return out


def after(code, age):
    """`age`: operations counted by lgkmcnt since the last LDS write that may be
    under way, it included (0: none).  (age at the end, at a barrier)"""
    barrier = 0
    for ins in code:
        op = ins[0]
        if op.startswith("ds_"):
            lane = op.startswith(("ds_read", "ds_bpermute", "ds_permute", "ds_swizzle"))
            age = (age and min(age + 1, LIMIT)) if lane else 1
        elif op.startswith(("s_load", "s_buffer_load", "flat_")):
            age = age and min(age + 1, LIMIT)
        elif op == "s_waitcnt":
            w = re.search(r"lgkmcnt\((\d+)\)", " ".join(ins))
            if w and age > int(w.group(1)):
                age = 0
        elif op == "s_barrier":
            barrier = barrier or age
    return age, barrier


def unwaited(blocks):
    """labels of the blocks with a barrier that an LDS write may pass"""
    at = {b: i for i, (b, _) in enumerate(blocks)}
    age, todo = {0: 0}, [0]
    while todo:
        i = todo.pop()
        code = blocks[i][1]
        end, _ = after(code, age[i])
        to = [at[c[1]] for c in code if c[0].startswith(("s_cbranch", "s_branch")) and c[1] in at]
        if i + 1 < len(blocks) and not any(c[0] in ("s_branch", "s_endpgm") for c in code):
            to.append(i + 1)
        for j in to:
            # the latest write of either path
            new = min((a for a in (age.get(j, 0), end) if a), default=0)
            if j not in age or new != age[j]:
                age[j] = new
                todo.append(j)
    return [blocks[i][0] for i in age if after(blocks[i][1], age[i])[1]]


def test_the_rule_itself():
    loop = "f:\n ds_write_b32 v0, v1\n s_waitcnt lgkmcnt(0)\n.LBB0_1:\n s_barrier\n%s" \
           " ds_write_b32 v0, v1\n s_cbranch_scc1 .LBB0_1\n s_endpgm\n"
    assert unwaited(functions(loop % "")["f"]) == [".LBB0_1"]
    waits = loop.replace("s_cbranch", "s_waitcnt vmcnt(0) lgkmcnt(0)\n s_cbranch") % ""
    assert unwaited(functions(waits)["f"]) == []
    one = "f:\n ds_write_b32 v0, v1\n ds_read_b32 v2, v3\n s_waitcnt lgkmcnt(%d)\n s_barrier\n"
    assert unwaited(functions(one % 1)["f"]) == []
    assert unwaited(functions(one % 2)["f"]) == [""]


def test_lds_writes_are_waited_for(tmp_path):
    flags = [f for f in B.HIP_FLAGS if f != "-Wall"]

    def compiled(src):
        out = str(tmp_path / (os.path.basename(src) + ".s"))
        subprocess.run(["hipcc", *flags, "--cuda-device-only", "-S", src, "-o", out], check=True,
                       capture_output=True)
        with open(out) as f:
            return f.read()

    srcs = sorted(glob.glob(os.path.join(B.CSRC, "*.hip")), key=os.path.getsize, reverse=True)
    with ThreadPoolExecutor(4) as pool:
        texts = list(pool.map(compiled, srcs))
    barriers, bad = 0, []
    for src, text in zip(srcs, texts):
        barriers += text.count("s_barrier")
        for name, blocks in functions(text).items():
            bad += [(os.path.basename(src), name, b) for b in unwaited(blocks)]
    assert barriers > 100  # (the assembly was read)
    assert not bad, bad

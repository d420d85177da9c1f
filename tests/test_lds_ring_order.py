"""The fp32 products keep a ring of LDS blocks per wave, without barriers: a step reads the next block
and copies a new one over the block whose operands it holds.  Such a copy is not ordered behind LDS
reads in flight, so the reads of a step have to be waited for before the copies of the next one.  What
a run does not show (a copy takes longer than a read, nearly always) the compiled code does: on every
path, an LDS read behind a copy is preceded by a wait for all reads before it."""
import os
import re
import subprocess

from paper_2305_12213_amd import build

RING = 20     # copies of the smallest ring: so many without a matrix instruction fill it, unread so far


def kernels_of(asm):
    """{name: [instructions and labels]} of the functions of an assembly listing."""
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name and re.match(r"\.LBB\w+:|\t[a-z]", line):
            out[name].append(line.split(";")[0].strip())
        elif name and line.startswith(".Lfunc_end"):
            name = None
    return {k: v for k, v in out.items() if "s_endpgm" in v}


def unordered_reads(lines):
    """LDS reads that some path reaches from a copy without a wait for the reads before that copy."""
    label_at = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    state = {0: (False, 0)}      # instruction -> (copy since the last wait, copies since the last MFMA)
    todo, bad = [0], set()
    while todo:
        i = todo.pop()
        dirty, run = state[i]
        l = lines[i]
        if l.startswith("s_waitcnt") and "lgkmcnt(0)" in l:
            dirty = False
        elif l.startswith("global_load_lds"):
            dirty, run = True, run + 1
        elif l.startswith("v_mfma"):
            run = 0
        elif l.startswith("ds_read") and dirty and run < RING:
            bad.add((i, l))
        after = [] if l.startswith(("s_endpgm", "s_branch")) else [i + 1]
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m:
            after.append(label_at[m.group(1)])
        for j in after:
            old = state.get(j)
            new = (dirty, run) if old is None else (dirty or old[0], min(run, old[1]))
            if new != old:
                state[j] = new
                todo.append(j)
    return sorted(bad)


def test_ring_slots_are_copied_into_after_their_reads(tmp_path):
    out = str(tmp_path / "gemm_f32.s")
    subprocess.run(["hipcc", *build.HIP_FLAGS, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "gemm_f32.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = kernels_of(f.read())
    assert len(kernels) == 5, list(kernels)     # forward / input gradient, two tile counts; weight gradient
    for name, lines in kernels.items():
        assert any(l.startswith("ds_read") for l in lines) and any(l.startswith("global_load_lds") for l in lines)
        assert not unordered_reads(lines), (name, unordered_reads(lines)[:4])

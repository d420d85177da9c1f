"""The fp32 products keep a ring of LDS blocks per wave, without barriers: a step reads the next block
and copies a new one over the block whose operands it holds.  Such a copy is not ordered behind LDS
reads in flight, so the reads of a step have to be waited for before the copies of the next one.  What
a run does not show (a copy takes longer than a read, nearly always) the compiled code does: on every
path, an LDS read behind a copy is preceded by a wait for all reads before it.  Where the waves of a workgroup share
a ring, what is copied over after a barrier was read by others before it: no wave arrives with reads in flight."""
import os
import re
import subprocess

import pytest

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


def is_copy(l):
    """Memory -> LDS without registers."""
    return l.startswith("global_load_lds") or l.startswith("buffer_load_dwordx4") and l.endswith("lds")


def walk(lines, start, step):
    """Follows every path: step(state, index, line) gives the state behind an instruction.  A state is a pair
    (something may be the case, the smallest count)."""
    label_at = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    state, todo = {0: start}, [0]
    while todo:
        i = todo.pop()
        l = lines[i]
        new = step(state[i], i, l)
        after = [] if l.startswith(("s_endpgm", "s_branch")) else [i + 1]
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m:
            after.append(label_at[m.group(1)])
        for j in after:
            old = state.get(j)
            both = new if old is None else (new[0] or old[0], min(new[1], old[1]))
            if both != old:
                state[j] = both
                todo.append(j)


def unordered_reads(lines):
    """LDS reads that some path reaches from a copy without a wait for the reads before that copy."""
    bad = set()

    def step(state, i, l):
        dirty, run = state       # copy since the last wait, copies since the last matrix instruction
        if l.startswith("s_waitcnt") and "lgkmcnt(0)" in l:
            dirty = False
        elif is_copy(l):
            dirty, run = True, run + 1
        elif l.startswith("v_mfma"):
            run = 0
        elif l.startswith("ds_read") and dirty and run < RING:
            bad.add((i, l))
        return dirty, run

    walk(lines, (False, 0), step)
    return sorted(bad)


def reads_in_flight_at_barriers(lines):
    """Barriers that some path reaches with LDS reads that it has not waited for."""
    bad = set()

    def step(state, i, l):
        pending, _ = state
        if l.startswith("s_waitcnt") and "lgkmcnt(0)" in l:
            pending = False
        elif l.startswith("ds_read"):
            pending = True
        elif l.startswith("s_barrier") and pending:
            bad.add((i, l))
        return pending, 0

    walk(lines, (False, 0), step)
    return sorted(bad)


def compiled(source, tmp_path):
    out = str(tmp_path / (source + ".s"))
    subprocess.run(["hipcc", *build.HIP_FLAGS, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return kernels_of(f.read())


@pytest.mark.parametrize("source,n", [
    ("gemm_f32.hip", 5),          # forward / input gradient, two tile counts; weight gradient
    ("gemm_f32_head.hip", 1),     # the last forward product with the loss
])
def test_ring_slots_are_copied_into_after_their_reads(source, n, tmp_path):
    kernels = compiled(source, tmp_path)
    assert len(kernels) == n, list(kernels)
    for name, lines in kernels.items():
        assert any(l.startswith("ds_read") for l in lines) and any(l.startswith("global_load_lds") for l in lines)
        assert not unordered_reads(lines), (name, unordered_reads(lines)[:4])


@pytest.mark.parametrize("source,which,n", [
    ("gemm_small.hip", "", 5),    # forward, with the loss, input gradient; weight gradients, past the caches or not
    ("gemm_lines.hip", "", 6),    # forward and input gradient, three shapes of tiles
    ("conv_wgrad.hip", "conv_wgrad_rows", 2),     # one or two groups of waves
    ("conv_wgrad.hip", "conv_wgrad_layers_rows", 2),      # ... for layers that share a launch
    ("conv_resident.hip", "", 4),                 # with and without mask and addend
])
def test_shared_rings_are_read_before_their_barriers(source, which, n, tmp_path):
    kernels = {k: v for k, v in compiled(source, tmp_path).items() if which in k}
    assert len(kernels) == n, list(kernels)
    for name, lines in kernels.items():
        assert any(l.startswith("ds_read") for l in lines) and any(is_copy(l) for l in lines)
        assert any(l.startswith("s_barrier") for l in lines)
        assert not reads_in_flight_at_barriers(lines), (name, reads_in_flight_at_barriers(lines)[:4])


def test_a_removed_wait_is_found(tmp_path):
    # the checks themselves, on listings with every wait for LDS taken out
    def without_waits(lines):
        return [l for l in lines if not (l.startswith("s_waitcnt") and "lgkmcnt" in l)]
    for lines in compiled("gemm_f32_head.hip", tmp_path).values():
        assert unordered_reads(without_waits(lines))
    for source in ("gemm_small.hip", "gemm_lines.hip"):
        for lines in compiled(source, tmp_path).values():
            assert reads_in_flight_at_barriers(without_waits(lines))

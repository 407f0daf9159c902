"""The projections whose activations go straight into the LDS wait for them by count: loads retire in the order in
which they were issued, so "at most N in flight" means that everything older has arrived - provided that every chunk
really issued the number of loads the count was made for.  The weight loads among them are ordinary loads, which a
compiler may leave out where nothing uses their value; the step would then read activations that are still on their
way, now and then.  Here the compiled kernels are walked, every path from the first request to the last wait, and at
every barrier the loads in flight have to be whole chunks, and none that the step behind the barrier reads."""
import os
import re
import subprocess

import pytest

from paper_2604_13519_amd import binding
from paper_2604_13519_amd.build import build_library

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def lds_loads(name):
    """LDS loads of one chunk in a wave; None: not a kernel that waits by count."""
    m = re.search(r"k_gemm_rows_bf16ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
    if m:
        mt, cs, kw, _ = map(int, m.groups())
        return -(-2 * mt * kw // 8)                         # two planes of mt x kw KiB over 8 waves
    m = re.search(r"k_gemm_few_bf16ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
    if m:
        mt, _, cs, kw, kc, _, _ = map(int, m.groups())
        return -(-2 * mt * (kc // 32) // (cs * kw))
    return None


def parse(text):
    """{kernel: [(address, event)]}: L / G a load into LDS / registers, "spill", ("wait", n), "barrier", "store", "end", ("jump", target, conditional)."""
    kernels, cur, start = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            start, cur = int(m.group(1), 16), kernels.setdefault(m.group(2), [])
            continue
        m = re.match(r"^\s+(\S+)(.*?)//\s*([0-9A-F]+):", line)
        if not m or cur is None:
            continue
        op, args, at = m.group(1), m.group(2), int(m.group(3), 16)
        if op.startswith("global_load_lds"):
            ev = "L"
        elif op.startswith("scratch_"):
            ev = "spill"
        elif re.match(r"(global|flat|buffer)_load", op):
            ev = "G"
        elif re.match(r"(global|flat|buffer)_(store|atomic)", op):
            ev = "store"
        elif op == "s_waitcnt":
            n = re.search(r"vmcnt\((\d+)\)", args)
            if not n:
                continue
            ev = ("wait", int(n.group(1)))
        elif op == "s_barrier":
            ev = "barrier"
        elif op == "s_endpgm":
            ev = "end"
        elif op.startswith("s_cbranch") or op == "s_branch":
            ev = ("jump", start + int(re.search(r"<\S+?\+0x([0-9a-f]+)>", line).group(1), 16), op != "s_branch")
        else:
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), line
            continue
        cur.append((at, ev))
    return kernels


def check(events, lds):
    """Walks every path.  State: the memory accesses in flight, oldest first (a load of a chunk as the number of chunks
    requested after its own, anything else as -1: it only makes a wait stricter), the LDS loads the newest chunk has so
    far, and by how many chunks the requests lead the barriers.  Returns the number of barriers met with loads in flight."""
    addr = [a for a, _ in events]
    first_at = lambda target: next(i for i, a in enumerate(addr) if a >= target)  # noqa: E731
    todo, seen, met = [(0, (), 0, 0)], set(), set()
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        i, flight, have, lead = state
        ev = events[i][1]
        if ev == "end" or ev == "store":                    # the results: nothing is requested from here on
            assert all(f < 0 for f in flight), "loads in flight at the first store"
            continue
        if ev == "L" and have in (0, lds):                  # a chunk begins
            flight, have, lead = tuple(f + 1 if f >= 0 else f for f in flight) + (0,), 1, lead + 1
        elif ev in ("L", "G"):
            flight, have = flight + (0 if have else -1,), have + (ev == "L")
        elif ev == "spill":
            flight = flight + (-1,)
        elif ev == "barrier":
            oldest = max([f for f in flight if f >= 0], default=-1)
            assert oldest < lead - 1 or oldest < 0, "the chunk behind a barrier has not arrived"
            if oldest >= 0:
                met.add(i)
            lead = max(lead - 1, 0)
        elif ev[0] == "wait":
            flight = flight[len(flight) - min(ev[1], len(flight)):]
        assert len(flight) < 256 and lead < 16, "requests without a wait"
        if isinstance(ev, tuple) and ev[0] == "jump":
            todo.append((first_at(ev[1]), flight, have, lead))
            if not ev[2]:
                continue
        todo.append((i + 1, flight, have, lead))
    return len(met)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no " + OBJDUMP)
    if not os.path.exists(binding.LIB_PATH):
        build_library(verbose=False)
    d = tmp_path_factory.mktemp("code")
    lib = os.path.join(str(d), "lib.so")
    os.symlink(binding.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=str(d), check=True, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(os.listdir(str(d))):
        if "gfx950" in f:
            text = subprocess.run([OBJDUMP, "-d", f], cwd=str(d), check=True, stdout=subprocess.PIPE, text=True).stdout
            found.update((k, v) for k, v in parse(text).items() if lds_loads(k))
    return found


def test_every_chunk_requests_what_the_waits_count(kernels):
    assert sum("k_gemm_rows_bf16" in k for k in kernels) == 45
    assert sum("k_gemm_few_bf16" in k for k in kernels) >= 20
    for name, events in kernels.items():
        try:
            n = check(events, lds_loads(name))
        except AssertionError as e:
            raise AssertionError("%s: %s" % (name, e))
        two_slots = re.search(r"k_gemm_rows_bf16ILi[78]ELi2ELi4E", name)          # these wait for all they have requested
        assert two_slots if n == 0 else not two_slots, name + ": %d barriers met with loads in flight" % n


def test_the_walk_notices_a_missing_load():
    """A ring of three slots, two loads into LDS and one into registers a chunk, with and without one weight load of the last trip."""
    def ring(loop_regs):
        ev = (["L", "L", "G"] * 2 + [("wait", 3), "barrier", "L", "L"] + ["G"] * loop_regs + [("jump", 6, True), ("wait", 3), "barrier", ("wait", 0), "barrier", "store"])
        return list(enumerate(ev))
    assert check(ring(1), 2) >= 2
    with pytest.raises(AssertionError):
        check(ring(0), 2)

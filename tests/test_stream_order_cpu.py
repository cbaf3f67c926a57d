"""The order of a plan's work on several streams, read from the runtime calls
the library makes (tests/c_stream_order.c stands in for the runtime): a launch
reads a pointer table only after the copy that filled it, a table is refilled
only after the launches that read it, on whichever streams these are, and the
events that say so release to system scope."""

import os
import shutil
import subprocess

import pytest

import paper_2609_25442_amd as wb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DISABLE_SYSTEM_FENCE = 0x20000000  # hipEventDisableSystemFence


@pytest.fixture(scope="module")
def client(tmp_path_factory):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    libdir = os.path.dirname(os.path.abspath(wb.LIB_PATH))
    exe = str(tmp_path_factory.mktemp("order") / "c_stream_order")
    subprocess.run([cc, "-std=gnu11", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c_stream_order.c"), "-o", exe,
                    "-L", libdir, "-l:" + os.path.basename(wb.LIB_PATH), "-Wl,-rpath," + libdir,
                    "-Wl,-rpath-link," + os.path.join(rocm, "lib")], check=True, capture_output=True, text=True)
    return exe


def _run(client, steps):
    out = subprocess.run([client, *steps], check=True, capture_output=True, text=True, timeout=60).stdout
    return [line.split() for line in out.splitlines()]


STEPS = [("A0", "B0"), ("A0", "B0", "A0", "B0"), ("A0", "B1", "B0", "A1"),
         ("A0", "A1", "A2", "A3", "B4", "B5", "A0", "B1", "A4", "B0"),
         ("A0", "B1", "C2", "A3", "B4", "C5", "C4", "A5", "B0", "C0", "A0")]


@pytest.mark.parametrize("steps", STEPS, ids="-".join)
def test_ordering_events_release_to_system_scope(client, steps):
    lines = _run(client, steps)
    flags = {e[1]: int(e[2], 16) for e in lines if e[0] == "event"}
    waited = {e[-1] for e in lines if e[0] in ("wait", "hostwait")}
    assert waited and all(not flags[e] & DISABLE_SYSTEM_FENCE for e in waited)


@pytest.mark.parametrize("steps", STEPS, ids="-".join)
def test_tables_are_copied_and_read_in_order(client, steps):
    """Every step's launch comes after the copy of its set and every refill after
    the launches that read the slot, by stream order or recorded events."""
    lines = _run(client, steps)
    at = [i for i, e in enumerate(lines) if e[0] == "step"]
    assert len(at) == len(steps)

    seen = {}       # event -> calls known to be complete when it has fired
    stream = {}     # stream -> calls known to be complete before its next call
    table, reads, fills, where = {}, {}, {}, {}

    for n, (a, b) in enumerate(zip(at, at[1:] + [len(lines)])):
        s, want = steps[n][0], steps[n][1]
        refill = [e for e in lines[a:b] if e[0] == "copy"]
        assert len(refill) <= 1 and sum(e[0] == "launch" for e in lines[a:b]) >= 1
        slot = refill[0][2] if refill else where[want]
        assert refill or table[slot] == want
        for i in range(a + 1, b):
            e = lines[i]
            if e[0] == "hostwait":
                continue
            assert e[1] == s
            done = stream.setdefault(s, set())
            if e[0] == "wait":
                done |= seen.get(e[2], set())
            elif e[0] == "record":
                seen[e[2]] = set(done)
            elif e[0] == "copy":
                assert reads.get(slot, set()) <= done, "a table is refilled under a launch that reads it"
                table[slot], where[want], fills[slot], reads[slot] = want, slot, i, set()
                done.add(i)
            elif e[0] == "launch":
                assert fills[slot] in done, "a launch reads a table before its copy"
                reads[slot].add(i)
                done.add(i)

"""Single-launch mode: the code of the attention kernels waits for the stores of partial rows before it counts a
delivery.

A workgroup may reduce rows that other workgroups of the same launch have stored, as soon as their deliveries are
counted.  A barrier does not wait for a wave's global stores on this target, so every wave has to, ahead of the
barrier behind which one of them counts.  No output shows a missing wait reliably; the code of the library as
built does: on its control-flow graph no path may lead from a device-coherent store (`sc1`) without an
`s_waitcnt vmcnt(0)`
 * to a count of arrivals, or
 * to a barrier from which a count is reached before another barrier, without a store of rows in between (the
   barrier that lets wave 0 count for the whole workgroup; a wave that runs a task on its own passes its
   barrier, stores, waits and counts).
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_17694_amd.binding import LIB_PATH

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def functions(listing):
    """name -> instructions (address, text, branch target or None)"""
    out, name, base = {}, None, 0
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
        if m:
            base, name = int(m.group(1), 16), m.group(2)
            out[name] = []
            continue
        m = re.match(r"^\t(.*?)\s*// ([0-9A-F]{12}): ", line)
        if m and name:
            to = re.search(r"<\S+?\+0x([0-9a-f]+)>$", line)
            target = base + int(to.group(1), 16) if to else base if line.endswith(f"<{name}>") else None
            out[name].append((int(m.group(2), 16), m.group(1).strip(), target))
    return out


def unwaited(ins):
    """(stores, counts, counts reached with a store unacknowledged, barriers of counts, those reached with one)"""
    index = {a: i for i, (a, _, _) in enumerate(ins)}
    succ = []
    for i, (_, text, target) in enumerate(ins):
        op = text.split()[0]
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "calls are not followed"
        if op == "s_endpgm":
            succ.append([])
        elif op == "s_branch":
            succ.append([index[target]])
        else:
            succ.append([i + 1] if i + 1 < len(ins) else [])
            if op.startswith("s_cbranch"):
                succ[i].append(index[target])
    every = range(len(ins))
    store = [re.match(r"global_store\S* .*\bsc1\b", t) is not None for _, t, _ in ins]
    wait = [t.startswith("s_waitcnt") and "vmcnt(0)" in t for _, t, _ in ins]
    barrier = [t.startswith("s_barrier") for _, t, _ in ins]
    # arrivals: a returning add at a per-lane address (the run-time queue's counters have a scalar base)
    count = [re.match(r"global_atomic_add v\d+, v\[\d+:\d+\], v\d+, off sc0", t) is not None for _, t, _ in ins]

    def reach(starts, stop):
        seen, work = set(), list(starts)
        while work:
            i = work.pop()
            if i not in seen:
                seen.add(i)
                if not stop[i]:
                    work += succ[i]
        return seen

    dirty = reach([s for i in every if store[i] for s in succ[i]], wait)
    gates = []
    for i in every:
        if barrier[i]:
            free = reach(succ[i], barrier)
            behind_stores = reach([s for j in free if store[j] for s in succ[j]], barrier)
            if any(count[j] and j not in behind_stores for j in free):
                gates.append(i)
    counts = [i for i in every if count[i]]
    return sum(store), len(counts), [i for i in counts if i in dirty], gates, [i for i in gates if i in dirty]


def test_every_wave_waits_for_its_stores(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    shutil.copy(LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    (image,) = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    listing = subprocess.run([OBJDUMP, "-d", image], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
    checked = 0
    for name, ins in functions(listing).items():
        if "pac_kernel" not in name or not name.endswith("ELb1EEEvNS_9PacParamsE"):     # without single-launch code
            continue
        stores, counts, early, gates, open_gates = unwaited(ins)
        assert stores and counts == 2 and gates, name            # by a workgroup, by a wave on its own
        assert not early, f"{name}: a delivery is counted with stores of rows in flight"
        assert not open_gates, f"{name}: a wave passes the barrier ahead of a count with stores of rows in flight"
        checked += 1
    assert checked == 12                # two data types, three head dimensions, two forms

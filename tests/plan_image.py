"""What a plan uploads to the GPU, read on the host: the planner compiled with g++ behind a small probe."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

import paper_2505_17694_amd.binding as B
from workloads import build_paged_kv

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2505_17694_amd", "csrc")

# DevTask of planner.hpp
RECORD = np.dtype([(n, np.int32) for n in ("page_off", "kv_len", "q_off", "n_req", "part_row_base", "solo_run", "flags", "single_req")])
LAYOUT = ("slot_recs", "slot_off", "num_slots", "queue_off", "queue_recs", "num_entries", "packs", "single_parts",
          "schedule", "fused", "makespan", "part_rows")


@functools.lru_cache(maxsize=None)
def _probe():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan_image.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(HERE, "plan_image.cpp"), os.path.join(CSRC, "planner.cpp"), "-o", so], check=True)
        lib = ctypes.CDLL(so)
    lib.image_blob.restype = ctypes.c_void_p
    lib.image_bytes.restype = ctypes.c_int64
    return lib


def rows_through(part_rows, kv_heads, head_dim):
    """(rows with tasks to follow, last rows): whether the two-launch kernels write them through to memory."""
    bits = _probe().image_rows_through(part_rows, kv_heads, head_dim)
    return bool(bits & 1), bool(bits & 2)


def plan_image(f, head, num_slots=0, split_align=0, max_rows=0, share=1, fixed_slices=0, schedule=0, fused=0,
               extensions=0, refreshed_len=None, paged=None):
    """The layout words, the packs and the task records of the plan, by slot and by queue entry."""
    lib = _probe()
    paged = paged if paged is not None else build_paged_kv(f, head, 3)
    a = {k: np.ascontiguousarray(v, np.int32) for k, v in (
        ("parent", f.parent), ("node_len", f.node_len), ("req_node", f.req_node),
        ("page_off", paged.node_page_off), ("pages", paged.page_ids))}
    off = words = None
    if getattr(f, "req_mask_off", None) is not None:
        off, words = np.ascontiguousarray(f.req_mask_off, np.int32), np.ascontiguousarray(f.req_mask, np.uint32)
    tree = B.codec_tree(len(f.parent), B._ptr(a["parent"]), B._ptr(a["node_len"]), len(f.req_node), B._ptr(a["req_node"]),
                        B._ptr(a["page_off"]), B._ptr(a["pages"]),
                        B._ptr(off) if off is not None else None,
                        B._ptr(words, ctypes.c_uint32) if words is not None else None)
    cfg = B.codec_head_config(head.num_q_heads, head.num_kv_heads, head.head_dim, head.dtype, head.page_size, head.scale)
    opt = B.codec_plan_options(num_slots, split_align, max_rows, share, None, fixed_slices, schedule, fused, extensions)
    grown = None if refreshed_len is None else np.ascontiguousarray(refreshed_len, np.int32)
    st = lib.image_plan(ctypes.byref(tree), ctypes.byref(cfg), ctypes.byref(opt), B._ptr(grown) if grown is not None else None)
    assert st == B.CODEC_OK, B.codec_status_string(st)
    v = (ctypes.c_int64 * len(LAYOUT))()
    lib.image_layout(v)
    out = dict(zip(LAYOUT, list(v)))
    n = out["packs"]
    packs, slot_off, slot_packs = np.zeros((n, 5), np.int64), np.zeros(out["num_slots"] + 1, np.int32), np.zeros(n, np.int32)
    lib.image_packs(packs.ctypes.data_as(ctypes.c_void_p), B._ptr(slot_off), slot_packs.ctypes.data_as(ctypes.c_void_p))
    out["packs"] = [dict(zip(("first", "step", "tiles", "rows", "cost"), p)) for p in packs.tolist()]
    out["pack_slots"] = [slot_packs[a:b].tolist() for a, b in zip(slot_off, slot_off[1:])] if n else []
    blob = np.ctypeslib.as_array(ctypes.cast(lib.image_blob(), ctypes.POINTER(ctypes.c_uint8)), (lib.image_bytes(),)).copy()

    def ints(at, n):
        return blob[at:at + 4 * n].view(np.int32)

    out["bytes"] = len(blob)
    out["slot_off"] = ints(out["slot_off"], out["num_slots"] + 1)
    out["queue_off"] = ints(out["queue_off"], out["num_entries"] + 1)
    for recs, offs in (("slot_recs", "slot_off"), ("queue_recs", "queue_off")):
        at = out[recs]
        out[recs] = blob[at:at + RECORD.itemsize * int(out[offs][-1])].view(RECORD)
    return out


def row_stores(f, head, **opts):
    """How a plan in two launches stores the rows of its dense and packed tasks, walked as the kernel walks its lists:
    bytes of partial rows, and per kind ("early": with tasks to follow in the workgroup, "last") the number of such
    tasks and whether their rows are written through."""
    im = plan_image(f, head, **opts)
    assert not im["fused"] and not im["single_parts"]
    group = head.num_q_heads // head.num_kv_heads
    queued = im["schedule"] == 1
    fetching = queued and im["num_entries"] > im["num_slots"]
    recs, off = (im["queue_recs"], im["queue_off"]) if queued else (im["slot_recs"], im["slot_off"])
    count = {"early": 0, "last": 0}
    for a, b in zip(off, off[1:]):
        for i in range(a, b):
            dense = int(recs[i]["n_req"]) * group > 16 if head.head_dim == 128 else recs[i]["flags"] & 4
            if dense:
                count["early" if i + 1 < b or fetching else "last"] += 1
    early, last = rows_through(im["part_rows"], head.num_kv_heads, head.head_dim)
    return {"bytes": im["part_rows"] * head.num_kv_heads * head.head_dim * 4, "early": (count["early"], early), "last": (count["last"], last), "image": im}

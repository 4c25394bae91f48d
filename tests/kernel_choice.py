"""Which kernels the library launches, seen without a GPU: a process of its own loads fake_hip.cpp in the place of the HIP
runtime and the library behind it, plans, "uploads" and decodes.  PyTorch, which has a runtime of its own, stays out of
that process: plans are handed over as arrays."""
import ctypes
import functools
import os
import pickle
import re
import subprocess
import sys
import tempfile
import types

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2505_17694_amd")


def case(f, paged, head, **opts):
    """What the other process needs of a plan."""
    masks = None if getattr(f, "req_mask_off", None) is None else (f.req_mask_off, f.req_mask)
    return dict(tree=[np.asarray(a) for a in (f.parent, f.node_len, f.req_node, paged.node_page_off, paged.page_ids)],
                masks=masks, head=(head.num_q_heads, head.num_kv_heads, head.head_dim, head.dtype, head.page_size, head.scale),
                pool=(paged.num_pages, paged.page_stride, paged.token_stride, paged.head_stride), opts=opts)


@functools.lru_cache(maxsize=None)
def _fake():
    _fake.folder = tempfile.TemporaryDirectory(prefix="codec-fake-hip-")        # goes with the process
    so = os.path.join(_fake.folder.name, "fake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


def launches(cases):
    """Per case, the kernels of one decode, of the partial attention alone and of the reduction alone, each a list of
    (name, template arguments, (grid x, y, z, threads of a block)); the plan's longest list, tasks and makespan."""
    return _ask("decode", cases)


def reduction_status(forms):
    """Status of a reduction launch for each (head_dim, split_waves), and the kernels it launched."""
    return _ask("reduction", forms)


def _ask(what, items):
    done = subprocess.run([sys.executable, os.path.abspath(__file__), what, _fake()], input=pickle.dumps(items),
                          stdout=subprocess.PIPE, check=True)
    return pickle.loads(done.stdout)


def _parse(lines):
    out = []
    for line in lines.decode().splitlines():
        name, *dims = line.split(" ")
        m = re.match(r"_ZN5codec(?:12_GLOBAL__N_1)?(\d+)", name)
        kernel = name[m.end():m.end() + int(m.group(1))]
        args = tuple(int(x) for x in re.findall(r"L[ib](\d+)E", name[m.end() + int(m.group(1)):]))
        out.append((kernel, args, tuple(int(x) for x in dims)))
    return out


def _main():
    what, so = sys.argv[1:]
    items = pickle.loads(sys.stdin.buffer.read())
    fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)             # ahead of the runtime that the library is linked to
    fake.fake_launches.restype = ctypes.c_char_p
    sys.modules["torch"] = None                                 # the binding does without it
    pkg = types.ModuleType("codec_binding")
    pkg.__path__ = [PKG]
    sys.modules["codec_binding"] = pkg
    from codec_binding import binding as B
    out = []
    if what == "reduction":
        launch = ctypes.cast(B._lib["_ZN5codec12launch_mergeERKNS_11MergeParamsEiiPv"], ctypes.c_void_p)
        for head_dim, waves in items:
            status = fake.fake_reduction(launch, head_dim, waves)
            out.append((status, _parse(fake.fake_launches())))
    for c in items if what == "decode" else ():
        o = dict(dict(num_slots=0, split_align=0, max_rows=0, share=1, cost_table=None, fixed_slices=0, schedule=0, extensions=0,
                      fused=0), **c["opts"])
        masks = c["masks"] if c["masks"] is not None else (None, None)
        st, plan = B.codec_plan_create(*c["tree"], *c["head"], o["num_slots"], o["split_align"], o["max_rows"], o["share"],
                                       o["cost_table"], o["fixed_slices"], o["schedule"], o["extensions"], o["fused"], *masks)
        assert st == B.CODEC_OK, st
        assert B.codec_plan_upload(plan, 4096, B.codec_plan_device_bytes(plan), 0) == B.CODEC_OK
        ws = B.codec_plan_workspace_bytes(plan)
        fake.fake_launches()
        seen = []
        for call in (lambda: B.codec_decode_attention(plan, 4096, 4096, 4096, *c["pool"], 4096, 4096, ws, 0),
                     lambda: B.codec_partial_attention(plan, 4096, 4096, 4096, *c["pool"], 4096, ws, 0),
                     lambda: B.codec_partial_reduction(plan, 4096, ws, 4096, 0)):
            assert call() == B.CODEC_OK
            seen.append(_parse(fake.fake_launches()))
        _, view = B.codec_plan_export(plan)
        out.append(dict(decode=seen[0], attention=seen[1], reduction=seen[2], tasks=len(view["tasks"]), makespan=view["makespan"],
                        longest=int(np.max(np.diff(view["req_part_off"])))))
        B.codec_plan_destroy(plan)
    sys.stdout.buffer.write(pickle.dumps(out))


if __name__ == "__main__":
    _main()

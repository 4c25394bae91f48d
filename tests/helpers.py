"""Test-side plumbing: logical views of paged K/V, written independently of the oracle."""
import numpy as np
import torch

from workloads import Forest, bits_to_float64, concat_forests, two_level_forest, unshared_forest, DTYPE_BF16, DTYPE_FP16


def token_slot(w, node, t):
    """(page, in-page slot) of logical token t of a node."""
    p = w.paged
    return int(p.page_ids[p.node_page_off[node] + t // p.page_size]), t % p.page_size


def pool_row(pool, w, page, slot, kvh):
    return pool[page, slot, kvh] if w.paged.layout == "thd" else pool[page, kvh, slot]


def request_context(w, r, kvh):
    """Concatenated (K, V) float64 [N_r, d] of request r for one KV head, root first: the tokens of the
    nodes on its path, without those of its last node that its visibility mask (if any) hides."""
    ks, vs = [], []
    f = w.forest
    words = None
    if getattr(f, "req_mask_off", None) is not None and f.req_mask_off[r + 1] > f.req_mask_off[r]:
        words = [int(x) for x in f.req_mask[f.req_mask_off[r]:f.req_mask_off[r + 1]]]
    for node in f.path(r):
        for t in range(int(f.node_len[node])):
            if words is not None and node == int(f.req_node[r]) and not (words[t // 32] >> (t % 32)) & 1:
                continue
            page, slot = token_slot(w, node, t)
            ks.append(pool_row(w.k_pool, w, page, slot, kvh))
            vs.append(pool_row(w.v_pool, w, page, slot, kvh))
    K = torch.stack(ks).to(torch.float64).numpy()
    V = torch.stack(vs).to(torch.float64).numpy()
    return K, V


def set_token(w, node, t, kvh, k_row=None, v_row=None):
    page, slot = token_slot(w, node, t)
    if k_row is not None:
        pool_row(w.k_pool, w, page, slot, kvh)[:] = torch.as_tensor(k_row).to(w.k_pool.dtype)
    if v_row is not None:
        pool_row(w.v_pool, w, page, slot, kvh)[:] = torch.as_tensor(v_row).to(w.v_pool.dtype)


def q_float64(w):
    return w.q.to(torch.float64).numpy()


# Packed row tiles of divided nodes: (channels, query heads, KV heads, requests per node, most rows of a pack with
# slices and a last tile smaller than the others or not).  64 channels: four, two and one waves per row group;
# 256 channels: one and two row tiles per wave.
DIVIDED_PACKS = [(64, 8, 2, 16, 64, False), (64, 8, 2, 32, 128, False), (64, 8, 2, 64, 256, False), (64, 4, 4, 41, 41, True),
                 (64, 12, 4, 43, 120, False), (64, 4, 4, 150, 150, True), (256, 8, 2, 16, 64, False),
                 (256, 8, 2, 32, 128, False), (256, 12, 4, 27, 81, True)]
DIVIDED_PACKS_OPTS = [{"num_slots": 2, "split_align": 32, "fixed_slices": 3},
                      {"num_slots": 2, "schedule": 1, "split_align": 64, "fixed_slices": 4},
                      {"num_slots": 2, "fused": 1, "fixed_slices": 2}]


def divided_packs_forest(requests):
    f = two_level_forest(33, [43] * requests)
    for n in (97, 513, 1000):
        f = concat_forests(f, two_level_forest(n, [5 + n % 40] * requests))
    return f


# Partial rows of dense (128 channels) and packed tasks, written through to memory or not: (channels, query heads, KV
# heads, requests per node, node lengths, slices per node, rows with tasks to follow written through or not, last rows).
# Every request ends at a node of many slices, so that wide tasks come first and last in a workgroup; 43 and 41 rows and
# their multiples leave a smaller last tile.
ROW_STORES = [
    (128, 32, 8, 43, (1000, 700, 300, 97), 12, True, False), (128, 16, 4, 43, (1000, 700, 300, 97), 12, True, True),
    (128, 12, 12, 43, (1000, 700, 300, 97), 12, True, True), (128, 8, 2, 43, (1000, 700, 300, 97), 12, False, True),
    (128, 32, 8, 43, (1000, 700), 5, False, False), (128, 16, 4, 43, (1000, 700), 4, False, True),
    (128, 32, 1, 13, (1000, 700), 4, False, True),
    (64, 32, 8, 43, (1000, 700, 300, 97), 12, True, False), (64, 16, 4, 43, (1000, 700, 300, 97), 30, True, True),
    (64, 12, 12, 41, (1000, 1000, 700, 300, 97), 30, True, True), (64, 80, 20, 23, (1000, 700), 11, True, True),
    (64, 8, 2, 43, (1000, 700, 300, 97), 16, False, True), (64, 32, 8, 43, (1000, 700), 11, False, False),
    (64, 8, 2, 43, (1000, 700), 16, False, True),
    (256, 16, 8, 43, (1000, 700, 300, 97), 8, True, False), (256, 8, 4, 43, (1000, 700, 300, 97), 8, True, True),
    (256, 12, 12, 41, (1000, 700, 300), 8, True, True), (256, 32, 4, 43, (1000, 700), 4, True, True),
    (256, 8, 2, 43, (1000, 700, 300, 97), 6, False, True),
    (256, 16, 8, 43, (1000, 700), 5, False, False), (256, 8, 4, 43, (1000, 700), 4, False, True)]
ROW_STORES_OPTS = [{"num_slots": 3}, {"num_slots": 2, "schedule": 1}]


def row_stores_forest(requests, lens):
    return Forest(np.full(len(lens), -1), np.array(lens), np.repeat(np.arange(len(lens)), requests))


# 32 requests of eight heads on one KV head end at a node of this many slices of one block (64 channels)
LONG_DIVISIONS = [32767, 32768]


def long_division_forest(slices):
    return Forest(np.array([-1]), np.array([32 * slices]), np.zeros(32, np.int64))


# Stream tasks that go round the KV heads in two launches ([token][head] pools): (channels, query heads, KV heads, data
# type, nodes, requests per node, requests below a shared node, form of the attention kernel: 0 stream tasks only, 1 all
# task shapes).  Contexts of up to 2300 tokens are cut in two: teams of waves and single-wave runs; 24 rows of 64 channels
# are two row tiles; the shared node brings dense tasks (128 channels) or, with 64, packed row tiles.  GOING_ROUND: all
# beside a shared node, in the form for all task shapes.
ROTATING = [(128, 32, 8, DTYPE_BF16, 60, 1, 0, 0), (128, 32, 8, DTYPE_FP16, 60, 1, 0, 0), (128, 28, 4, DTYPE_FP16, 120, 1, 0, 0),
            (128, 9, 3, DTYPE_BF16, 140, 2, 0, 0), (64, 16, 8, DTYPE_BF16, 60, 1, 0, 0), (64, 16, 8, DTYPE_FP16, 60, 1, 0, 0),
            (64, 64, 8, DTYPE_FP16, 60, 3, 0, 0), (64, 32, 4, DTYPE_BF16, 110, 3, 0, 0),
            (128, 32, 8, DTYPE_FP16, 60, 1, 40, 1), (64, 64, 8, DTYPE_FP16, 30, 1, 64, 1), (64, 64, 8, DTYPE_BF16, 30, 1, 64, 1)]
GOING_ROUND = [(128, 32, 8, 110), (128, 28, 4, 200), (128, 9, 3, 280), (64, 16, 8, 110), (64, 12, 12, 90)]
GOING_ROUND_OPTS = [{"num_slots": 1}, {"num_slots": 2}, {"num_slots": 3, "schedule": 1}]
ROTATING_OPTS = [{"num_slots": 2, "fixed_slices": 2}, {"num_slots": 3, "fixed_slices": 2, "schedule": 1}]


def going_round_forest(leaves):
    return concat_forests(two_level_forest(300, [17 + 13 * (i % 9) for i in range(leaves)]), unshared_forest([2200, 33, 700]))


def rotating_forest(nodes, requests, below):
    lens = [17 + (389 * i) % 2290 for i in range(nodes)]
    f = Forest(np.full(nodes, -1), np.array(lens), np.repeat(np.arange(nodes), requests))
    return concat_forests(f, two_level_forest(700, [33 + 17 * (i % 5) for i in range(below)])) if below else f

"""The ways an attention pass is cut into workgroups, against the fp64 oracle:
one, two, four and eight key groups and stream mode, one layer at a time, at
sizes where a cut can go wrong (a cache that ends inside a tile or on its edge,
fewer tiles than key groups, a last query tile of a few rows), and the mass
sweep cut along the query rows.  The bars are the parity suite's: outputs to
bf16, W to 1e-3."""
import numpy as np
import pytest
import torch

from oracle import hermes_oracle as orc
from paper_2601_14724_amd import streaming, workloads as wk

from _parity import check_o, f64, gen, oracle_caches, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # name, Hq, Hkv, d, T0, C
    ("one_group_empty_cache", 4, 4, 64, 0, 33),
    ("two_groups_edge_of_tile", 28, 4, 128, 128, 784),
    ("two_groups_one_past_it", 28, 4, 128, 641, 784),
    ("four_groups_d128", 28, 4, 128, 1000, 300),
    ("four_groups_d64", 14, 2, 64, 900, 784),
    ("eight_groups_fewer_tiles", 8, 2, 64, 257, 1),
    ("eight_groups_d64", 14, 2, 64, 1024, 196),
    ("eight_groups_d128", 6, 3, 128, 191, 65),
    ("stream_d64", 14, 2, 64, 4000, 300),
    ("stream_d128", 28, 4, 128, 6144, 196),
    ("stream_g9", 9, 1, 128, 2001, 64),
]


@pytest.mark.parametrize("name,Hq,Hkv,d,T0,C", SHAPES)
def test_append_cuts_match_oracle(name, Hq, Hkv, d, T0, C):
    """Two layers appended one by one, then in one call: outputs and W."""
    wl = wk.custom(name, 300 + C % 97, 2, Hq, Hkv, d, T0, C, (T0 + C, T0 + C), anchor_period=37)
    say(f"[cuts] {name}: Hq={Hq} Hkv={Hkv} d={d} T0={T0} C={C}")
    caches, chunks = gen(wl)
    kv = streaming.make_cache(wl, caches=caches, force_scores=True, layer_class=[2, 2])
    t = streaming.chunk_tensors({k: np.stack([c[k] for c in chunks]) for k in ("q", "k", "v")} |
                                {"pos": chunks[0]["pos"]})
    single = torch.stack([kv.append(t["q"][l], t["k"][l], t["v"][l], t["pos"], layer=l) for l in range(2)])
    w = [kv.w[l][:T0 + C].cpu().numpy().astype(np.float64) for l in range(2)]
    kv.rewind()
    both = kv.append(t["q"], t["k"], t["v"], t["pos"])
    oc = oracle_caches(caches)
    for l in range(2):
        k, v = f64(chunks[l]["k"]), f64(chunks[l]["v"])
        o, wr = orc.chunk_attention(f64(chunks[l]["q"]), oc[l].k.reshape(T0, Hkv, d), oc[l].v.reshape(T0, Hkv, d), k, v)
        check_o(single[l].float().cpu().numpy(), o, f"[cuts] {name} layer {l} alone")
        check_o(both[l].float().cpu().numpy(), o, f"[cuts] {name} layer {l} of two")
        for x in (w[l], kv.w[l][:T0 + C].cpu().numpy().astype(np.float64)):
            rel = float((np.abs(x - wr) / wr).max())
            assert rel <= 1e-3, f"{name} layer {l}: mass off by {rel}"
    kv.close()

"""The ways an attention pass is cut into workgroups, against the fp64 oracle:
one, two, four and eight key groups, stream mode and split mode, at sizes where a cut can go wrong (a cache that ends inside a tile or on its edge,
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
    ("four_groups_short_cache_d128", 6, 3, 128, 191, 65),
    ("eight_groups_or_split_two_groups_d64", 14, 2, 64, 4000, 300),
    ("split_two_groups_or_stream_d128", 28, 4, 128, 6144, 196),
    ("split_four_groups_d128", 28, 4, 128, 2600, 130),
    ("split_eight_groups_64_rows_d64", 14, 2, 64, 2300, 64),
    ("split_eight_groups_d128", 9, 1, 128, 2001, 64),
    ("eight_groups_200_rows_d64", 8, 1, 64, 1900, 200),
    ("eight_groups_one_row_d64", 12, 3, 64, 1300, 1),
    ("stream_d64", 14, 2, 64, 3000, 1200),
]


QUERIES = [
    # name, layers, Hq, Hkv, d, lengths of the caches, rows
    ("one_row_d64", 2, 2, 2, 64, (129, 1000), 1),
    ("one_row_of_seven_heads", 3, 28, 4, 128, (700, 2048, 2049), 1),
    ("32_packed_rows", 2, 8, 2, 128, (1, 1500), 8),
    ("33_packed_rows", 2, 33, 3, 64, (640, 3000), 3),
    ("64_packed_rows", 2, 8, 1, 128, (1023, 2500), 8),
    ("65_packed_rows", 2, 13, 1, 128, (900, 2047), 5),
    ("128_packed_rows", 2, 4, 4, 64, (500, 1601), 128),
    ("129_packed_rows", 2, 3, 1, 128, (900, 4000), 43),
    ("four_groups_unequal", 2, 28, 4, 128, (700, 4001), 64),
]


# Each instance of the attention kernel: a pass that takes it (tests/test_plan_host.py
# holds the library to the cut named here).
CUTS = [
    # cut, d, Hq, Hkv, lengths of the caches, rows
    ("plain 1", 64, 16, 16, (130,) * 6, 1),
    ("plain 2", 64, 16, 16, (130,) * 6, 130),
    ("plain 4", 64, 16, 16, (130,) * 6, 64),
    ("plain 8", 64, 4, 4, (257,), 1),
    ("split 2", 64, 28, 4, (2600,), 300),
    ("split 4", 64, 14, 2, (6001,), 196),
    ("split 8", 64, 9, 1, (2001,), 16),
    ("four waves, 32 rows", 64, 4, 4, (2001,), 1),
    ("four waves, 64 rows", 64, 9, 1, (2600,), 5),
    ("four waves, 128 rows", 64, 9, 1, (2600,), 8),
    ("stream", 64, 9, 1, (5000,), 5),
    ("plain 1", 128, 4, 4, (130,), 1),
    ("plain 2", 128, 16, 16, (130,) * 6, 130),
    ("plain 4", 128, 9, 1, (130,), 16),
    ("plain 8", 128, 4, 4, (257,), 1),
    ("split 2", 128, 9, 1, (2600,) * 6, 64),
    ("split 4", 128, 9, 1, (500,), 16),
    ("split 8", 128, 9, 1, (1300,), 16),
    ("four waves, 32 rows", 128, 4, 4, (641,), 1),
    ("four waves, 64 rows", 128, 9, 1, (641,), 5),
    ("four waves, 128 rows", 128, 9, 1, (641,), 8),
    ("stream", 128, 9, 1, (5000,), 5),
]
PROMPTS = [
    # the same for passes for the row LSE alone
    ("plain 1", 64, 4, 4, (130,), 1),
    ("plain 2", 64, 16, 16, (130,) * 6, 130),
    ("plain 4", 64, 32, 8, (130,) * 6, 43),
    ("plain 8", 64, 4, 4, (257,), 1),
    ("plain 1", 128, 4, 4, (130,), 1),
    ("plain 2", 128, 16, 16, (130,) * 6, 130),
    ("plain 4", 128, 9, 1, (130,), 16),
    ("plain 8", 128, 4, 4, (257,), 1),
    ("four waves, 32 rows", 128, 4, 4, (2600,), 1),
    ("stream", 64, 9, 1, (5000,), 5),
]


@pytest.mark.parametrize("cut,d,Hq,Hkv,lens,rows", CUTS)
def test_every_cut_of_a_query_matches_oracle(cut, d, Hq, Hkv, lens, rows):
    from paper_2601_14724_amd import hermes as H
    L = len(lens)
    say(f"[cuts] {cut}: {Hq}/{Hkv} d={d} lens={lens} rows={rows}")
    init, host = [], []
    for l, n in enumerate(lens):
        wl = wk.custom("cut", 800 + rows, L, Hq, Hkv, d, n, 1, (n,) * L, query_len=rows, anchor_period=29)
        c, q = wk.gen_cache(wl, l), wk.gen_query(wl, l)
        host.append((c, q))
        init.append((streaming.bf16_tensor(c["k"], "cuda"), streaming.bf16_tensor(c["v"], "cuda"),
                     torch.from_numpy(c["pos"]).cuda()))
    kv = H.HermesKV(L, Hq, Hkv, d, list(lens), rows, init=init)
    out = kv.query(*(streaming.bf16_tensor(np.stack([q[k] for _, q in host]), "cuda") for k in ("q", "k", "v")))
    for l, (c, q) in enumerate(host):
        o, _ = orc.chunk_attention(f64(q["q"]), f64(c["k"]), f64(c["v"]), f64(q["k"]), f64(q["v"]), want_w=False)
        check_o(out[l].float().cpu().numpy(), o, f"[cuts] {cut} layer {l}")
    kv.close()


@pytest.mark.parametrize("cut,d,Hq,Hkv,lens,rows", PROMPTS)
def test_every_cut_of_a_prompt_matches_oracle(cut, d, Hq, Hkv, lens, rows):
    """W of every cached token (the last one appended just before) from the
    prompt's rows."""
    from paper_2601_14724_amd import hermes as H
    L = len(lens)
    say(f"[cuts] prompt {cut}: {Hq}/{Hkv} d={d} lens={lens} rows={rows}")
    init, host = [], []
    for l, n in enumerate(lens):
        wl = wk.custom("prompt", 900 + rows, L, Hq, Hkv, d, n, 1, (n,) * L, query_len=rows, anchor_period=29)
        c, q = wk.gen_cache(wl, l), wk.gen_query(wl, l)
        host.append((c, q))
        init.append((streaming.bf16_tensor(c["k"][:-1], "cuda"), streaming.bf16_tensor(c["v"][:-1], "cuda"),
                     torch.from_numpy(c["pos"][:-1]).cuda()))
    kv = H.HermesKV(L, Hq, Hkv, d, list(lens), rows, init=init, layer_class=[2] * L, scoring_mode=H.SCORE_GUIDANCE)
    last = {k: streaming.bf16_tensor(np.stack([c[k][-1:] for c, _ in host]), "cuda") for k in ("k", "v")}
    q1 = torch.zeros(L, 1, Hq, d, dtype=torch.bfloat16, device="cuda")
    kv.append(q1, last["k"], last["v"], torch.from_numpy(host[0][0]["pos"][-1:]).cuda())
    kv.guidance(*(streaming.bf16_tensor(np.stack([q[k] for _, q in host]), "cuda") for k in ("q", "k", "v")))
    torch.cuda.synchronize()
    for l, (c, q) in enumerate(host):
        _, w = orc.chunk_attention(f64(q["q"]), f64(c["k"]), f64(c["v"]), f64(q["k"]), f64(q["v"]))
        n = lens[l]
        rel = float((np.abs(kv.w[l][:n].cpu().numpy().astype(np.float64) - w[:n]) / w[:n]).max())
        assert rel <= 1e-3, f"{cut} layer {l}: mass off by {rel}"
    kv.close()


@pytest.mark.parametrize("name,L,Hq,Hkv,d,lens,rows", QUERIES)
def test_query_cuts_match_oracle(name, L, Hq, Hkv, d, lens, rows):
    """Queries over caches of unequal lengths, all layers in one call and one
    by one."""
    from paper_2601_14724_amd import hermes as H
    say(f"[cuts] query {name}: {Hq}/{Hkv} d={d} lens={lens} rows={rows}")
    init, host = [], []
    for l, n in enumerate(lens):
        wl = wk.custom(name, 400 + rows, L, Hq, Hkv, d, n, 1, (n,) * L, query_len=rows, anchor_period=29)
        c, q = wk.gen_cache(wl, l), wk.gen_query(wl, l)
        host.append((c, q))
        init.append((streaming.bf16_tensor(c["k"], "cuda"), streaming.bf16_tensor(c["v"], "cuda"),
                     torch.from_numpy(c["pos"]).cuda()))
    kv = H.HermesKV(L, Hq, Hkv, d, [max(lens)] * L, rows, init=init)
    t = {k: streaming.bf16_tensor(np.stack([q[k] for _, q in host]), "cuda") for k in ("q", "k", "v")}
    both = kv.query(t["q"], t["k"], t["v"])
    for l, (c, q) in enumerate(host):
        o, _ = orc.chunk_attention(f64(q["q"]), f64(c["k"]), f64(c["v"]), f64(q["k"]), f64(q["v"]), want_w=False)
        check_o(both[l].float().cpu().numpy(), o, f"[cuts] query {name} layer {l} of {L}")
        alone = kv.query(t["q"][l], t["k"][l], t["v"][l], layer=l)
        check_o(alone.float().cpu().numpy(), o, f"[cuts] query {name} layer {l} alone")
    kv.close()


@pytest.mark.parametrize("rows", [64, 100])
def test_queries_on_several_streams_match_oracle(rows):
    """Layers queried at the same time on four streams of one context: three have
    a room for partial rows, the fourth takes the shared one (64 rows) or another
    cut."""
    from paper_2601_14724_amd import hermes as H
    L, Hq, Hkv, d, n = 4, 14, 2, 64, 3000
    say(f"[cuts] queries of {rows} rows on {L} streams")
    init, host = [], []
    wl = wk.custom("streams", 500 + rows, L, Hq, Hkv, d, n, 1, (n,) * L, query_len=rows, anchor_period=29)
    for l in range(L):
        c, q = wk.gen_cache(wl, l), wk.gen_query(wl, l)
        host.append((c, q))
        init.append((streaming.bf16_tensor(c["k"], "cuda"), streaming.bf16_tensor(c["v"], "cuda"),
                     torch.from_numpy(c["pos"]).cuda()))
    kv = H.HermesKV(L, Hq, Hkv, d, [n] * L, rows, init=init)
    t = {k: streaming.bf16_tensor(np.stack([q[k] for _, q in host]), "cuda") for k in ("q", "k", "v")}
    out = torch.zeros_like(t["q"])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(L)]
    for _ in range(4):
        for l, s in enumerate(streams):
            with torch.cuda.stream(s):
                kv.query(t["q"][l], t["k"][l], t["v"][l], layer=l, out=out[l])
    torch.cuda.synchronize()
    for l, (c, q) in enumerate(host):
        o, _ = orc.chunk_attention(f64(q["q"]), f64(c["k"]), f64(c["v"]), f64(q["k"]), f64(q["v"]), want_w=False)
        check_o(out[l].float().cpu().numpy(), o, f"[cuts] query of {rows} rows, stream {l}")
    kv.close()


def test_captured_query_beside_a_longer_one_matches_oracle():
    """A recorded one-row query replayed on one stream while 100-row queries run
    on another: the recorded one's partial rows have a room that the other stream
    never writes."""
    from paper_2601_14724_amd import hermes as H
    Hq, Hkv, d, n, rows = 28, 4, 128, 4096, (100, 1)
    say("[cuts] captured query of 1 row beside queries of 100")
    init, host = [], []
    for l in range(2):
        wl = wk.custom("captured", 600 + l, 2, Hq, Hkv, d, n, 1, (n,) * 2, query_len=rows[l], anchor_period=29)
        c, q = wk.gen_cache(wl, l), wk.gen_query(wl, l)
        host.append((c, q))
        init.append((streaming.bf16_tensor(c["k"], "cuda"), streaming.bf16_tensor(c["v"], "cuda"),
                     torch.from_numpy(c["pos"]).cuda()))
    kv = H.HermesKV(2, Hq, Hkv, d, [n] * 2, 100, init=init)
    t = [{k: streaming.bf16_tensor(q[k], "cuda") for k in ("q", "k", "v")} for _, q in host]
    out = [torch.zeros(40, *t[l]["q"].shape, dtype=torch.bfloat16, device="cuda") for l in range(2)]
    short = torch.zeros_like(t[1]["q"])
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        kv.query(t[0]["q"], t[0]["k"], t[0]["v"], layer=0, out=out[0][0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=b):
        kv.query(t[1]["q"], t[1]["k"], t[1]["v"], layer=1, out=short)
    for i in range(40):
        with torch.cuda.stream(a):
            kv.query(t[0]["q"], t[0]["k"], t[0]["v"], layer=0, out=out[0][i])
        with torch.cuda.stream(b):
            graph.replay()
            out[1][i].copy_(short)
    torch.cuda.synchronize()
    for l, (c, q) in enumerate(host):
        o, _ = orc.chunk_attention(f64(q["q"]), f64(c["k"]), f64(c["v"]), f64(q["k"]), f64(q["v"]), want_w=False)
        check_o(out[l][0].float().cpu().numpy(), o, f"[cuts] query of {rows[l]} rows")
        assert (out[l] == out[l][0]).all(), f"{rows[l]} rows: a pass differs from the first"
    kv.close()


def test_appends_on_four_streams_match_oracle():
    """Layers appended at the same time on four streams: three have a room for
    partial rows, the fourth runs another cut; outputs and W."""
    L, Hq, Hkv, d, T0, C = 4, 14, 2, 64, 3000, 196
    say(f"[cuts] appends of {C} rows on {L} streams")
    wl = wk.custom("append_streams", 700, L, Hq, Hkv, d, T0, C, (T0 + C,) * L, anchor_period=37)
    caches, chunks = gen(wl)
    kv = streaming.make_cache(wl, caches=caches, force_scores=True, layer_class=[2] * L)
    t = streaming.chunk_tensors({k: np.stack([c[k] for c in chunks]) for k in ("q", "k", "v")} |
                                {"pos": chunks[0]["pos"]})
    out = torch.zeros_like(t["q"])
    streams = [torch.cuda.Stream() for _ in range(L)]
    for _ in range(4):
        torch.cuda.synchronize()
        kv.rewind()
        for l, s in enumerate(streams):
            with torch.cuda.stream(s):
                kv.append(t["q"][l], t["k"][l], t["v"][l], t["pos"], layer=l, out=out[l])
    torch.cuda.synchronize()
    oc = oracle_caches(caches)
    for l in range(L):
        k, v = f64(chunks[l]["k"]), f64(chunks[l]["v"])
        o, wr = orc.chunk_attention(f64(chunks[l]["q"]), oc[l].k.reshape(T0, Hkv, d), oc[l].v.reshape(T0, Hkv, d), k, v)
        check_o(out[l].float().cpu().numpy(), o, f"[cuts] append on stream {l}")
        rel = float((np.abs(kv.w[l][:T0 + C].cpu().numpy().astype(np.float64) - wr) / wr).max())
        assert rel <= 1e-3, f"stream {l}: mass off by {rel}"
    kv.close()


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

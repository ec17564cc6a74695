"""The attention tiles at their edges: segments and windows that leave tiles of
1, 15, 16, 17, 63, 64 rows, every group size, both head dims, per-head masks,
and the library's own choice for a group of eight against the split kernels.

Tolerance of the outputs against fp64: the cut of p into three bf16 terms is
exact and the sums are fp32, so only the rounding of the bf16 output (half an
ulp: seven stored bits, so up to 2^-8 of the value) and fp32 sums of up to 400
products (400 * 2^-24 of the largest |V|, 4e-5 for |V| <= 1.7) remain."""
import numpy as np
import pytest
import torch

import _harness as H
import paper_2503_10571_amd as radar
from oracle import radar_oracle as orc

pytestmark = pytest.mark.gpu


def _inputs(cfg, seed, vmax=1.7):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    shape = (cfg.batch, cfg.n_kv_heads, cfg.capacity, cfg.head_dim)
    K = torch.randn(shape, generator=g, device="cuda").to(cfg.dtype)
    V = torch.randn(shape, generator=g, device="cuda").clamp(-vmax, vmax).to(cfg.dtype)
    q = torch.randn(cfg.batch, cfg.n_q_heads, cfg.head_dim, generator=g,
                    device="cuda").to(cfg.dtype)
    omega = torch.randn(cfg.n_features, cfg.head_dim, generator=g,
                        device="cuda").to(torch.bfloat16).float()
    return K, V, q, omega


def _close(out, ref, dtype):
    half_ulp = 2.0 ** -8 if dtype == torch.bfloat16 else 0.0
    bad = np.abs(out - ref) > half_ulp * np.abs(ref) * 1.01 + 4e-5
    assert not bad.any(), (np.argwhere(bad)[:4], out[bad][:4], ref[bad][:4])


@pytest.mark.parametrize("c,w", [(1, 1), (15, 17), (16, 63), (17, 64), (63, 65), (64, 16),
                                 (65, 130), (100, 3)])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("d,dtype", [(64, torch.bfloat16), (128, torch.bfloat16),
                                     (64, torch.float32), (128, torch.float32)])
def test_partial_tiles(c, w, G, d, dtype):
    t, n_sink = 3 + 6 * c + w, 3
    for per_head in (radar.GQA_UNION, radar.GQA_PER_HEAD):
        print(f"[case] attend c={c} w={w} G={G} d={d} {dtype} per_head={per_head}", flush=True)
        cfg = radar.Config(1, G, 1, d, 64, c, w, t + 70, dtype, n_sink, per_head)
        K, V, q, _ = _inputs(cfg, 7 * c + w)
        ws, n_cand = orc.window_split(t, c, w, n_sink)
        sel = torch.full((1, G, 3), -1, dtype=torch.int32, device="cuda")
        for h in range(G):
            ids = [(h * 5 + 1) % n_cand, (h * 3) % n_cand]
            sel[0, h, :2] = torch.tensor(ids, dtype=torch.int32)
        out = H.f64(radar.attend_selected(cfg, q, K, V, sel, t))
        own = [[int(s) for s in sel[0, h] if s >= 0] for h in range(G)]
        for h in range(G):
            ids = own[h] if per_head else [s for o in own for s in o]
            toks = orc.attended_tokens(ids, c, ws, t, n_sink)
            ref = orc.attend(H.f64(q[0, h]), H.f64(K[0, 0]), H.f64(V[0, 0]), toks)
            _close(out[0, h], ref, dtype)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_infinite_value(G, d):
    """An infinite V element in a tile without masked rows makes its output
    infinite, not NaN, although p has a single significant bit (all logits
    are equal: p = 1), so that its second and third term are 0."""
    cfg = radar.Config(1, G, 1, d, 64, 16, 128, 128, torch.bfloat16)
    K, V, q, _ = _inputs(cfg, 3)
    K.zero_()
    for t in (64, 128):
        print(f"[case] inf V G={G} d={d} t={t}", flush=True)
        v = V.clone()
        v[0, 0, 0, 5] = float("inf")
        v[0, 0, t - 1, 9] = float("-inf")
        sel = torch.full((1, G, 1), -1, dtype=torch.int32, device="cuda")
        out = radar.attend_selected(cfg, q, K, v, sel, t).float()
        assert bool((out[0, :, 5] == float("inf")).all())
        assert bool((out[0, :, 9] == float("-inf")).all())
        rest = [i for i in range(d) if i not in (5, 9)]
        ref = H.f64(v[0, 0, :t, rest]).mean(0)
        for h in range(G):
            _close(H.f64(out[0, h, rest]), ref, torch.bfloat16)


def _same_as_split(cfg, t, k, lens, want):
    """decode and append_decode by the library's own choice, which has to be
    `want` by its query and by the kernels that ran, against the forced split
    path: the same selections, scores, rows and summaries, outputs within
    their rounding."""
    K, V, q, omega = _inputs(cfg, 11)
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    kernel = {radar.PATH_SPLIT: "topk", radar.PATH_SELECT: "select", radar.PATH_SCORED: "scored"}
    res = {}
    for path in (radar.PATH_AUTO, radar.PATH_SPLIT):
        radar.set_decode_path(path)
        radar.profile_enable(True)
        try:
            takes = radar.decode_path(cfg, t, k)
            assert takes == (want if path == radar.PATH_AUTO else radar.PATH_SPLIT)
            sel = torch.empty(cfg.batch, cfg.n_q_heads, k, dtype=torch.int32, device="cuda")
            sc = torch.empty(cfg.batch, cfg.n_q_heads, k, device="cuda")
            out = radar.decode(cfg, q, K, V, omega, summ, t, k, selected=sel, scores=sc, lens=lens)
            ran = radar.profile_read()
            for p, name in kernel.items():
                assert ran[name][1] == (1 if p == takes else 0), (name, ran)
            K2, V2, summ2 = K.clone(), V.clone(), summ.clone()
            step = radar.append_decode(cfg, q, K2, V2, K[:, :, t].clone(), V[:, :, t].clone(),
                                       omega, summ2, t + 1, k, pos=lens)
            res[path] = (out, sel, sc, step, K2, V2, summ2)
        finally:
            radar.profile_enable(False)
            radar.profile_read()
            radar.set_decode_path(radar.PATH_AUTO)
    a, b = res[radar.PATH_AUTO], res[radar.PATH_SPLIT]
    for i in (1, 4, 5, 6):
        assert torch.equal(a[i], b[i]), i
    assert torch.equal(a[2].nan_to_num(-1.0), b[2].nan_to_num(-1.0))
    ulp = 2.0 ** -7 if cfg.dtype == torch.bfloat16 else 0.0
    for i in (0, 3):
        x, y = H.f64(a[i]), H.f64(b[i])
        assert np.array_equal(np.isnan(x), np.isnan(y))
        bad = np.abs(x - y) > ulp * np.abs(y) + 8e-5
        assert not bad.any()


OPTIONS = ["plain", "sinks", "per_head", "ragged", "no_candidates", "w0"]


def _route(opt, G, d, dtype, n=128):
    t = 1500 if opt != "no_candidates" else 60
    cfg = radar.Config(3, 2 * G, 2, d, n, 37, 0 if opt == "w0" else 90, t + 4, dtype,
                       5 if opt == "sinks" else 0,
                       radar.GQA_PER_HEAD if opt == "per_head" else radar.GQA_UNION)
    lens = torch.tensor([t, t // 2, 0], device="cuda") if opt == "ragged" else None
    return cfg, t, lens


@pytest.mark.parametrize("opt", OPTIONS)
@pytest.mark.parametrize("d", [64, 128])
def test_group_of_eight_route(opt, d):
    """The library's choice for a group of eight."""
    print(f"[case] g8 route {opt} d={d}", flush=True)
    cfg, t, lens = _route(opt, 8, d, torch.bfloat16)
    _same_as_split(cfg, t, 7, lens, radar.PATH_SCORED)


@pytest.mark.parametrize("opt", OPTIONS)
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_f32_d128_route(opt, G):
    """The library's choice for fp32 caches at d = 128: with one head these
    170 KB of Omega and summary rows make a light selection."""
    print(f"[case] fp32 route {opt} G={G}", flush=True)
    cfg, t, lens = _route(opt, G, 128, torch.float32, n=256)
    want = {1: radar.PATH_SELECT, 8: radar.PATH_SPLIT}.get(G, radar.PATH_SCORED)
    _same_as_split(cfg, t, 7, lens, want)


@pytest.mark.parametrize("G,n,want", [(2, 256, radar.PATH_SELECT), (1, 2048, radar.PATH_SPLIT)])
def test_f32_d128_idle_cus(G, n, want):
    """fp32 calls at d = 128 whose idle CUs leave much of the stream to the
    others: 9/16 as many pairs (one workgroup each) as CUs, of 3 MB or more, with
    few summary rows and with many."""
    print(f"[case] fp32 idle G={G} n={n}", flush=True)
    pairs = torch.cuda.get_device_properties(0).multi_processor_count * 9 // 16
    cfg = radar.Config(1, G * pairs, pairs, 128, n, 64, 60, 4104, torch.float32)
    _same_as_split(cfg, 4100, 40, None, want)


@pytest.mark.parametrize("n_cand,k", [(1025, 7), (2047, 256), (300, 256)])
@pytest.mark.parametrize("per_head", [radar.GQA_UNION, radar.GQA_PER_HEAD])
def test_group_of_eight_many_candidates(n_cand, k, per_head):
    """More candidates than the fused kernel takes, and the largest k."""
    print(f"[case] g8 n_cand={n_cand} k={k}", flush=True)
    t = 3 * n_cand + 5
    cfg = radar.Config(2, 16, 2, 128, 64, 3, 4, t + 2, torch.bfloat16, 0, per_head)
    _same_as_split(cfg, t, k, None, radar.PATH_SCORED)


@pytest.mark.parametrize("call", ["decode", "split", "append_decode", "exact", "given"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_more_tiles_than_partials(call, dtype):
    """A pair whose tiles, one per wave, would need more workgroups than a
    merge takes partials (a window of 4110 tiles; 4 waves, 1024 partials): its
    waves take several. The sums stay short: at most three tiles of 64 tokens
    per wave, four waves, and 32 partials per thread and 32 threads in the
    merge, so the 400 products of _close hold."""
    G, w = 8, 4110 * 64 - 5
    t = w + 300
    print(f"[case] wide attention {call} {dtype} t={t}", flush=True)
    cfg = radar.Config(1, G, 1, 64, 64, 64, w, t, dtype)
    K, V, q, omega = _inputs(cfg, 5)
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    ws, n_cand = orc.window_split(t, 64, w, 0)
    k = 2
    sel = torch.empty(1, G, k, dtype=torch.int32, device="cuda")
    if call == "append_decode":
        out = radar.append_decode(cfg, q, K, V, K[:, :, -1].clone(), V[:, :, -1].clone(), omega,
                                  summ, t, k, selected=sel)
    elif call == "exact":
        out = radar.decode_exact(cfg, q, K, V, t, k, selected=sel)
    elif call == "given":
        sel[:] = torch.arange(k, dtype=torch.int32) * 2
        out = radar.attend_selected(cfg, q, K, V, sel, t)
    else:
        radar.set_decode_path(radar.PATH_SPLIT if call == "split" else radar.PATH_AUTO)
        try:
            out = radar.decode(cfg, q, K, V, omega, summ, t, k, selected=sel)
        finally:
            radar.set_decode_path(radar.PATH_AUTO)
    toks = orc.attended_tokens([int(s) for s in sel.flatten().tolist()], 64, ws, t, 0)
    keys, vals = H.f64(K[0, 0]), H.f64(V[0, 0])
    for h in (0, G - 1):
        _close(H.f64(out[0, h]), orc.attend(H.f64(q[0, h]), keys, vals, toks), dtype)

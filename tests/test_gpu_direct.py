"""GPU parity of the prefill tiles that are copied straight to LDS and run the expand as further K tiles: sizes at the edges
of tiles, several tiles per workgroup, blocks whose adapters take one K tile, many and none, a captured launch, and an
adapter whose values are not finite."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, announce, rel_err, run_and_check
from paper_2602_24044_amd import binding as B
from paper_2602_24044_amd import workloads as wl
from paper_2602_24044_amd.runtime import Session, bf16_tensor_to_bits

pytestmark = pytest.mark.gpu

NAMES = ["direct_256x256x64_w4", "direct_256x192x64_w4", "direct_128x256x64_w4"]
TILES = [B.FUSED_VARIANTS[n] for n in NAMES]


def _expected(variant, on=True):
    return (["shrink", "expand_tiles"] if on else []) + ["gemm_fused_" + NAMES[TILES.index(variant)]]


def _launches(w, tuning=None, path=B.LORA_PATH_AUTO, gated=False):
    """Names of the launches of projection 0 (of the gated call of 0 and 1)."""
    sess = Session(w, path=path)
    try:
        for key, value in (tuning or {}).items():
            B.lora_set_tuning(sess.ctx, key, value)
        sess.load(w.resident)
        sess.bucket()
        sess.forward_glu(0, 1) if gated else sess.forward(0)
        return B.lora_last_launches(sess.ctx)
    finally:
        sess.close()


def _check(w, variant, **kw):
    """The tile that was asked for runs, and its results agree with the oracle."""
    tuning = {B.LORA_TUNE_FUSED_VARIANT: variant}
    assert _launches(w, tuning, B.LORA_PATH_FUSED) == _expected(variant, len(w.resident) > 0)
    run_and_check(w, path=B.LORA_PATH_FUSED, tuning=tuning, **kw)


def _runs(rng, n_tokens, n_ad, longest):
    """Whole prompts in token order, some without an adapter."""
    return np.repeat(rng.integers(-1, n_ad, size=n_tokens), rng.integers(1, longest + 1, size=n_tokens))[:n_tokens].astype(np.int32)


@pytest.mark.parametrize("variant", TILES)
@pytest.mark.parametrize("n_tokens,proj,mode,ranks", [
    (1, [(192, 8)], wl.BUCKET_SORTED, [64]),                                   # three K tiles, one row, one chunk of columns
    (129, [(256, 200), (256, 256)], wl.BUCKET_SORTED, [8, 16]),
    (256, [(192, 264)], wl.BUCKET_RUNS, [8]),
    (257, [(320, 520), (320, 72), (320, 192)], wl.BUCKET_RUNS, [8, 16, 32, 64]),
    (1030, [(192, 16392)], wl.BUCKET_RUNS, [16, 64]),                          # more tiles than CUs with every tile shape
])
def test_tile_edges(n_tokens, proj, mode, ranks, variant):
    rng = np.random.default_rng(n_tokens)
    ids = _runs(rng, n_tokens, 6, 90) if mode == wl.BUCKET_RUNS else rng.integers(-1, 6, size=n_tokens).astype(np.int32)
    w = wl.custom("direct_edges", n_tokens, proj, [f"p{k}" for k in range(len(proj))], 6, 64, mode, ids, {i: ranks[i % len(ranks)] for i in range(6)})
    _check(w, variant)


@pytest.mark.parametrize("row_tiles,cols", [(2, 66568), (4, 33800), (6, 22400), (8, 16648), (16, 8456), (17, 8200), (32, 4360)])
def test_every_tile_once_whatever_the_row_tiles(row_tiles, cols):
    # two rounds and more of 256 x 256 tiles; from round to round the deal turns by 0, 1 or 8 places.  The last block of rows has
    # twenty adapters, the others one or none
    n_tokens = row_tiles * 256 - 3
    ids = np.full(n_tokens, -1, dtype=np.int32)
    ids[:n_tokens // 3] = 0
    ids[-200:] = 1 + np.arange(200) // 10
    w = wl.custom("direct_deal", row_tiles, [(192, cols)], ["p"], 21, 16, wl.BUCKET_RUNS, ids, {i: 16 if i % 2 else 8 for i in range(21)})
    _check(w, TILES[0])


@pytest.mark.parametrize("variant", TILES)
def test_bias_and_packed_slices(variant):
    _check(wl.qwen_decode(shrink=8, n_tokens=300), variant, packed=True)


@pytest.mark.parametrize("variant", TILES)
def test_no_adapter_resident(variant):
    ids = np.full(300, -1, dtype=np.int32)
    w = wl.custom("direct_base", 2, [(256, 264), (256, 72)], ["p", "r"], 1, 8, wl.BUCKET_SORTED, ids, {0: 8}, resident=[])
    _check(w, variant)
    _check(w, variant, packed=True)


@pytest.mark.parametrize("n_ad", [0, 1, 40, 150])
def test_adapters_per_block(n_ad):
    # 300 tokens of so many adapters of rank 64 behind four K tiles of the backbone.  The sorted rows' two blocks hold one adapter
    # each (n_ad = 1), 34 and 7 (40) or 128 and 22 (150), and as many K tiles; n_ad = 0: no row has one, but one is resident
    ids = (np.arange(300) % max(n_ad, 1)).astype(np.int32) if n_ad else np.full(300, -1, dtype=np.int32)
    w = wl.custom("direct_adapters", n_ad, [(256, 264)], ["p"], max(n_ad, 1), 64, wl.BUCKET_SORTED, ids, {i: 64 for i in range(max(n_ad, 1))})
    for variant in TILES:
        _check(w, variant)


def _gated(w, tuning):
    adapters = len(w.resident) > 0
    announce(f"glu direct {w.name} T={w.T} proj={w.proj[0]}")
    sess = Session(w)
    try:
        B.lora_set_tuning(sess.ctx, B.LORA_TUNE_FUSED_VARIANT, tuning)
        sess.load(w.resident)
        sess.bucket()
        out = sess.forward_glu(0, 1)
        torch.cuda.synchronize()
        assert B.lora_last_launches(sess.ctx) == (["shrink", "expand_tiles"] if adapters else []) + ["gemm_glu_direct_256x256x64_w4"]
        h_ref = oracle.gated(w.x[0], w.W[0], w.W[1], w.token_ids, oracle.adapters_of(w, 0), oracle.adapters_of(w, 1))
        assert rel_err(bf16_tensor_to_bits(out), h_ref) <= TOL
    finally:
        sess.close()


@pytest.mark.parametrize("n_tokens,cols,ranks", [(1, 8, [16]), (255, 136, [8, 64]), (257, 1000, [16]), (1100, 8200, [8, 16, 32])])
def test_gated_tiles(n_tokens, cols, ranks):
    rng = np.random.default_rng(cols)
    w = wl.custom("direct_glu", cols, [(192, cols), (192, cols)], ["gate", "up"], 6, 64, wl.BUCKET_RUNS, _runs(rng, n_tokens, 6, 60),
                  {i: ranks[i % len(ranks)] for i in range(6)})
    _gated(w, TILES[0])


def test_gated_tiles_without_a_resident_adapter():
    w = wl.custom("direct_glu_base", 9, [(192, 520), (192, 520)], ["gate", "up"], 1, 8, wl.BUCKET_RUNS, np.full(300, -1, dtype=np.int32), {0: 8}, resident=[])
    _gated(w, TILES[0])


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("n_tokens,n_ad,rank,order", [
    (300, 4, 64, "turns"),                                # every row a run of its own, four adapters per block
    (513, 150, 16, "random"),                             # runs of one and two rows; most adapters come back
    (260, 256, 8, "turns"),                               # 256 runs in a block and none comes back; four come back in the next
    (512, 3, 64, "palindrome"),                           # 0 1 2 1 0, runs that cross the windows of 16 rows
])
def test_adapters_that_come_back(n_tokens, n_ad, rank, order, gated):
    rng = np.random.default_rng(n_ad)
    if order == "turns":
        ids = np.arange(n_tokens) % n_ad
    elif order == "palindrome":
        ids = np.repeat([0, 1, -1, 2, 1, 0], 37)
        ids = np.tile(ids, n_tokens // len(ids) + 1)[:n_tokens]
    else:
        ids = np.repeat(rng.integers(-1, n_ad, size=n_tokens), rng.integers(1, 3, size=n_tokens))[:n_tokens]
    proj = [(256, 264)] * (2 if gated else 1)
    w = wl.custom("direct_back", n_tokens, proj, ["gate", "up"][:len(proj)], n_ad, 64, wl.BUCKET_RUNS, ids.astype(np.int32), {i: rank if i % 5 else 8 for i in range(n_ad)})
    if gated:
        _gated(w, TILES[0])
    else:
        for variant in TILES:
            _check(w, variant)


def _gemm_ms(w, variant):
    sess = Session(w, path=B.LORA_PATH_FUSED)
    try:
        B.lora_set_tuning(sess.ctx, B.LORA_TUNE_FUSED_VARIANT, variant)
        sess.load(w.resident)
        sess.bucket()
        for _ in range(3):
            sess.forward(0)
        torch.cuda.synchronize()
        B.lora_profile_enable(sess.ctx, True)
        for _ in range(20):
            sess.forward(0)
        torch.cuda.synchronize()
        ms, count = B.lora_profile_collect(sess.ctx)["gemm_fused_" + NAMES[TILES.index(variant)]]
        return ms / count
    finally:
        sess.close()


@pytest.mark.parametrize("variant", TILES)
def test_adapters_that_come_back_are_expanded_once(variant):
    # the same four adapters of rank 64 token by token and as one prompt each: four K tiles of expand per block against one or two,
    # behind sixteen.  A K tile per run would be 256 of them
    ms = []
    for ids in (np.arange(1024) // 256, np.arange(1024) % 4):
        w = wl.custom("direct_once", 1, [(1024, 1024)], ["p"], 4, 64, wl.BUCKET_RUNS, ids.astype(np.int32), {i: 64 for i in range(4)})
        ms.append(_gemm_ms(w, variant))
    announce(f"one prompt each {ms[0] * 1e3:.1f} us, in turns {ms[1] * 1e3:.1f} us")
    assert ms[1] < 3.0 * ms[0]


def test_128_rows_take_their_own_adapters_of_the_block():
    # 256 rows of 128 adapters of rank 64: sorted, each half of the block has 64 of them (64 K tiles behind three), in turns both
    # have all
    ms = []
    for ids in (np.repeat(np.arange(128), 2), np.arange(256) % 128):
        w = wl.custom("direct_half", 1, [(192, 1024)], ["p"], 128, 64, wl.BUCKET_RUNS, ids.astype(np.int32), {i: 64 for i in range(128)})
        ms.append(_gemm_ms(w, B.FUSED_VARIANTS["direct_128x256x64_w4"]))
    announce(f"sorted {ms[0] * 1e3:.1f} us, in turns {ms[1] * 1e3:.1f} us")
    assert ms[0] < 0.75 * ms[1]


@pytest.mark.parametrize("n_tokens,order", [(400, "sorted"), (256, "sorted"), (390, "back")])
def test_128_rows_of_a_block(n_tokens, order):
    # halves whose first chunk is not a multiple of eight, without an adapter, and (RUNS) with an adapter of the other half
    if order == "sorted":
        ids = np.sort(np.random.default_rng(7).integers(-1, 90, size=n_tokens))
        ids[:40] = -1
    else:
        ids = np.concatenate([np.repeat(np.arange(13), 10)[:128], np.full(100, -1), np.repeat([5, 20, 11], 40), np.full(42, 20)])
    w = wl.custom("direct_half", n_tokens, [(256, 264)], ["p"], 90, 64, wl.BUCKET_RUNS, ids.astype(np.int32), {i: (8, 24, 64)[i % 3] for i in range(90)})
    _check(w, B.FUSED_VARIANTS["direct_128x256x64_w4"])


@pytest.mark.parametrize("n_tokens,cols,gated,kernel", [
    (1300, 4096, False, "gemm_fused_direct_128x256x64_w4"),
    (2100, 4104, False, "gemm_fused_direct_256x192x64_w4"),
    (2049, 28680, False, "gemm_fused_direct_256x256x64_w4"),
    (257, 28672, False, "gemm_fused_direct_256x256x64_w4"),
    (777, 14336, True, "gemm_glu_direct_256x256x64_w4"),
    (1025, 18944, True, "gemm_glu_direct_256x256x64_w4"),
])
def test_automatic_choice(n_tokens, cols, gated, kernel):
    # what runs for large batches of few adapters, and what the launch log calls it
    rng = np.random.default_rng(n_tokens)
    proj = [(192, cols)] * (2 if gated else 1)
    w = wl.custom("direct_auto", 4, proj, ["gate", "up"][:len(proj)], 2, 8, wl.BUCKET_RUNS, _runs(rng, n_tokens, 2, 90), {0: 8, 1: 8})
    assert _launches(w, gated=gated) == ["shrink", "expand_tiles", kernel]


STAGED = {"gemm_fused_direct_128x256x64_w4": "gemm_fused_staged_128x256x64_w8", "gemm_fused_direct_256x192x64_w4": "gemm_fused_staged_256x192x64_w8",
          "gemm_fused_direct_256x256x64_w4": "gemm_fused_staged_256x256x64_w8", "gemm_glu_direct_256x256x64_w4": "gemm_glu_staged_256x256x64_w8"}


@pytest.mark.parametrize("n_tokens,cols,gated,most,kernel", [
    # sorted, several rounds: 8 (1 + adapters / blocks) ranks of at most 0.45 of K = 192, gated twice as many of at most 0.4
    (2049, 28680, False, 78, "gemm_fused_direct_256x256x64_w4"),
    (1025, 18944, True, 15, "gemm_glu_direct_256x256x64_w4"),
    # a single round: 8 (gated 16) ranks of every adapter, of at most 0.5 of K
    (1300, 4096, False, 12, "gemm_fused_direct_128x256x64_w4"),
    (2100, 4104, False, 12, "gemm_fused_direct_256x192x64_w4"),
    (1025, 2048, True, 6, "gemm_glu_direct_256x256x64_w4"),
])
def test_sorted_batches_of_many_adapters_take_the_staged_tiles(n_tokens, cols, gated, most, kernel):
    proj = [(192, cols)] * (2 if gated else 1)
    for n_ad in (most, most + 1):
        ids = (np.arange(n_tokens) % n_ad).astype(np.int32)
        w = wl.custom("direct_many", 4, proj, ["gate", "up"][:len(proj)], n_ad, 8, wl.BUCKET_SORTED, ids, {i: 8 for i in range(n_ad)})
        assert _launches(w, gated=gated) == (["shrink", "expand_tiles", kernel] if n_ad == most else ["shrink", STAGED[kernel]]), n_ad


@pytest.mark.parametrize("max_rank,kernels", [(8, ["shrink", "expand_tiles", "gemm_fused_direct_128x256x64_w4"]),
                                              (64, ["shrink", "gemm_fused_staged_128x256x64_w8"])])
def test_expand_tables_that_do_not_fit_the_scratch(max_rank, kernels):
    # 20000 rows of bf16 shrink results, 0.3 or 2.6 MB, beside the tables in 1 MB of scratch for partial tiles
    w = wl.custom("direct_scratch", 4, [(192, 256)], ["p"], 2, max_rank, wl.BUCKET_RUNS, np.repeat([0, 1], 10000).astype(np.int32), {0: 8, 1: max_rank})
    sess = Session(w, split_k=1)
    try:
        sess.load(w.resident)
        sess.bucket()
        out = sess.forward(0)
        assert B.lora_last_launches(sess.ctx) == kernels
        y_ref = oracle.project(w.x[0], w.W[0], w.token_ids, oracle.adapters_of(w, 0))
        assert rel_err(bf16_tensor_to_bits(out), y_ref) <= TOL
    finally:
        sess.close()


@pytest.mark.parametrize("n_tokens,kernel", [(65532, "gemm_fused_direct_256x256x64_w4"), (65536, "gemm_fused_staged_256x256x64_w8")])
def test_output_of_four_gigabytes(n_tokens, kernel):
    w = wl.custom("direct_4g", 4, [(192, 32768)], ["p"], 1, 8, wl.BUCKET_RUNS, np.full(n_tokens, -1, dtype=np.int32), {0: 8}, resident=[])
    assert _launches(w) == [kernel]


@pytest.mark.parametrize("n_tokens,cols,gated,kernel", [
    (1300, 4096, False, "gemm_fused_direct_128x256x64_w4"),
    (2100, 4104, False, "gemm_fused_direct_256x192x64_w4"),
    (1025, 2056, True, "gemm_glu_direct_256x256x64_w4"),
])
def test_runs_of_few_and_many_adapters_on_one_captured_launch(n_tokens, cols, gated, kernel):
    # 60 resident adapters of rank 8: in token order a block of rows may hold one of them or all.  The launches of both kernels
    # are made and the block maps say which does the work: with more than 12 chunks per block (gated 6) the staged one
    rng = np.random.default_rng(12)
    few = np.repeat(np.arange(n_tokens // 100 + 1) % 60, 100)[:n_tokens]
    many = rng.integers(-1, 60, size=n_tokens)
    edge = np.concatenate([many[:256], np.full(n_tokens - 256, 3)])      # one block of many among blocks of one
    proj = [(192, cols)] * (2 if gated else 1)
    w = wl.custom("direct_or_staged", 5, proj, ["gate", "up"][:len(proj)], 60, 8, wl.BUCKET_RUNS, few.astype(np.int32), {i: 8 for i in range(60)})
    sess = Session(w)
    try:
        sess.load(w.resident)

        def step():
            sess.bucket()
            return sess.forward_glu(0, 1, out=sess.out[0]) if gated else sess.forward(0)

        step()
        assert B.lora_last_launches(sess.ctx) == ["shrink", "expand_tiles", kernel, STAGED[kernel]]
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step()
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            step()
        for rep, ids in enumerate((many, few, many, edge, few)):
            ids = ids.astype(np.int32)
            sess.ids.copy_(torch.from_numpy(ids).to(sess.device))
            sess.out[0].fill_(float("nan"))
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            if gated:
                y_ref = oracle.gated(w.x[0], w.W[0], w.W[1], ids, oracle.adapters_of(w, 0), oracle.adapters_of(w, 1))
            else:
                y_ref = oracle.project(w.x[0], w.W[0], ids, oracle.adapters_of(w, 0))
            assert rel_err(bf16_tensor_to_bits(sess.out[0]), y_ref) <= TOL, rep
    finally:
        sess.close()


@pytest.mark.parametrize("n_tokens", [1100, 300])
@pytest.mark.parametrize("variant", TILES)
def test_captured_launch_on_new_token_ids(variant, n_tokens):
    # every replay has other ids: blocks of few, many and no adapters behind each other, so that what a replay before left in
    # the expand's tables does not fit
    rng = np.random.default_rng(3)
    w = wl.custom("direct_graph", 3, [(256, 1032)], ["p"], 40, 32, wl.BUCKET_SORTED, rng.integers(-1, 40, size=n_tokens).astype(np.int32),
                  {i: 8 << (i % 3) for i in range(40)})
    sess = Session(w, path=B.LORA_PATH_FUSED)
    try:
        B.lora_set_tuning(sess.ctx, B.LORA_TUNE_FUSED_VARIANT, variant)
        sess.load(w.resident)
        sess.step()
        assert B.lora_last_launches(sess.ctx) == _expected(variant)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            sess.step()
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            sess.step()
        for rep, top in enumerate((40, 1, 40, 0, 6)):
            ids = rng.integers(-1, top, size=w.T).astype(np.int32)
            sess.ids.copy_(torch.from_numpy(ids).to(sess.device))
            sess.out[0].zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            y_ref = oracle.project(w.x[0], w.W[0], ids, oracle.adapters_of(w, 0))
            assert rel_err(bf16_tensor_to_bits(sess.out[0]), y_ref) <= TOL, rep
    finally:
        sess.close()


@pytest.mark.parametrize("variant", TILES)
def test_values_that_are_not_finite_stay_with_their_adapter(variant):
    # tokens of adapter 1 sit between those of 0 and 2; its B holds an infinity, which must reach its own 16-row windows only
    ids = np.repeat(np.arange(3, dtype=np.int32), 48)
    w = wl.custom("direct_inf", 1, [(192, 264)], ["p"], 3, 16, wl.BUCKET_RUNS, ids, {0: 16, 1: 16, 2: 8})
    outs = []
    for poison in (False, True):
        if poison:
            w.adapters[1].B[0][:, 3] = 0x7f80                  # + infinity in bf16
        sess = Session(w, path=B.LORA_PATH_FUSED)
        try:
            B.lora_set_tuning(sess.ctx, B.LORA_TUNE_FUSED_VARIANT, variant)
            sess.load(w.resident)
            sess.bucket()
            outs.append(sess.forward(0).clone())
            torch.cuda.synchronize()
        finally:
            sess.close()
    clean, poisoned = outs
    assert bool(torch.isfinite(clean).all())
    assert not bool(torch.isfinite(poisoned[48:96]).any())
    assert torch.equal(clean[:48], poisoned[:48]) and torch.equal(clean[96:], poisoned[96:])


@pytest.mark.parametrize("variant", TILES)
def test_values_that_are_not_finite_of_an_adapter_that_comes_back(variant):
    # adapters 0, 1, 0, 2, 1, 0 of three windows each in a block, adapter 1 with an infinity: its chunks lie between the others'
    ids = np.repeat(np.array([0, 1, 0, 2, 1, 0], dtype=np.int32), 48)
    w = wl.custom("direct_inf_back", 1, [(192, 264)], ["p"], 3, 16, wl.BUCKET_RUNS, ids, {0: 16, 1: 16, 2: 8})
    outs = []
    for poison in (False, True):
        if poison:
            w.adapters[1].B[0][:, 3] = 0x7f80
        sess = Session(w, path=B.LORA_PATH_FUSED)
        try:
            B.lora_set_tuning(sess.ctx, B.LORA_TUNE_FUSED_VARIANT, variant)
            sess.load(w.resident)
            sess.bucket()
            outs.append(sess.forward(0).clone())
            torch.cuda.synchronize()
        finally:
            sess.close()
    clean, poisoned = outs
    mine = torch.from_numpy(ids == 1).to(clean.device)
    assert bool(torch.isfinite(clean).all())
    assert not bool(torch.isfinite(poisoned[mine]).any())
    assert torch.equal(clean[~mine], poisoned[~mine])

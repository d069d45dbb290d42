"""GPU parity of every selectable GEMM kernel variant (lora_set_tuning) against the CPU oracle: the
automatic choice reaches only some of them at a given shape, the others stay reachable for tuning and must
compute the same result.  Small workloads with a ragged last tile, packed and single calls."""
import numpy as np
import pytest
import torch

from gpu_util import run_and_check
from paper_2602_24044_amd import binding as B
from paper_2602_24044_amd import workloads as wl
from paper_2602_24044_amd.runtime import Session

pytestmark = pytest.mark.gpu

FUSED_VARIANTS = sorted(B.FUSED_VARIANTS.values())
SPLIT_VARIANTS = sorted(B.SPLIT_VARIANTS.values())


def _launches(w, tuning=None, path=B.LORA_PATH_AUTO):
    """Names of the launches of projection 0."""
    sess = Session(w, path=path)
    try:
        for key, value in (tuning or {}).items():
            B.lora_set_tuning(sess.ctx, key, value)
        sess.load(w.resident)
        sess.bucket()
        sess.forward(0)
        return B.lora_last_launches(sess.ctx)
    finally:
        sess.close()


@pytest.mark.parametrize("variant", FUSED_VARIANTS)
def test_fused_variant_decode_and_prefill(variant):
    tuning = {B.LORA_TUNE_FUSED_VARIANT: variant}
    run_and_check(wl.config2(shrink=8, n_tokens=300), path=B.LORA_PATH_FUSED, tuning=tuning)
    run_and_check(wl.config3(shrink=8, n_req=6, len_div=8), path=B.LORA_PATH_FUSED, tuning=tuning, packed=True)


@pytest.mark.parametrize("variant", SPLIT_VARIANTS)
def test_split_variant_decode(variant):
    tuning = {B.LORA_TUNE_SPLIT_VARIANT: variant}
    run_and_check(wl.config2(shrink=8, n_tokens=300), path=B.LORA_PATH_SPLITK, tuning=tuning)
    run_and_check(wl.config4(shrink=8), path=B.LORA_PATH_SPLITK, split_k=3, tuning=tuning, packed=True)


@pytest.mark.parametrize("variant", [6, 7])
def test_whole_line_split_variants_short_k_ranges(variant):
    # 16 splits of a 512-wide K leave every workgroup fewer K tiles than the ring has stages
    tuning = {B.LORA_TUNE_SPLIT_VARIANT: variant}
    run_and_check(wl.config1(), path=B.LORA_PATH_SPLITK, split_k=16, tuning=tuning)
    run_and_check(wl.config1(), path=B.LORA_PATH_SPLITK, split_k=2, tuning=tuning)


@pytest.mark.parametrize("mode", [B.LORA_INLINE_SHRINK_OFF, B.LORA_INLINE_SHRINK_ON])
@pytest.mark.parametrize("variant", [8, 9, 10, 11])
def test_shrink_inside_the_fused_launch(mode, variant):
    # fused path up to 1024 tokens: the shrink by the first workgroups of the GEMM launch, or as a launch of its own;
    # two steps in a row (the launch leaves its counters at zero for the next one)
    tuning = {B.LORA_TUNE_INLINE_SHRINK: mode, B.LORA_TUNE_FUSED_VARIANT: variant}
    run_and_check(wl.config2(shrink=8, n_tokens=300), path=B.LORA_PATH_FUSED, tuning=tuning, packed=True)
    run_and_check(wl.config4(shrink=8), path=B.LORA_PATH_FUSED, tuning=tuning, packed=True)
    run_and_check(wl.qwen_decode(shrink=4, n_tokens=200), path=B.LORA_PATH_FUSED, tuning=tuning)


@pytest.mark.parametrize("path", [B.LORA_PATH_FUSED, B.LORA_PATH_SPLITK])
@pytest.mark.parametrize("n_tokens", [1, 31, 32, 33, 63, 64, 65])
def test_small_batch_tiles_and_their_edges(n_tokens, path):
    # 32- and 64-row tiles and the first size behind each.  K of gate|up is 512, 448 (shrink 8) and 2048 (shrink 2, where the
    # fused launch starts its column tiles at different places of K)
    run_and_check(wl.config2(shrink=8, n_tokens=n_tokens), path=path, packed=True)
    run_and_check(wl.qwen_decode(shrink=8, n_tokens=n_tokens), path=path)
    if n_tokens in (1, 33):
        run_and_check(wl.config2(shrink=2, n_tokens=n_tokens), path=path, packed=True)


@pytest.mark.parametrize("n_tokens,cols,kernel", [
    (1300, 4096, "gemm_fused_staged_128x256x64_w8"),        # 176 tiles: one round of two thirds of a 256 x 256 round
    (2100, 4104, "gemm_fused_staged_256x192x64_w8"),        # ragged last column tile, ragged last row tile
    (2049, 28680, "gemm_fused_staged_256x256x64_w8"),       # nine row tiles, the last with one row; XCD runs of unequal length
    (257, 28672, "gemm_fused_staged_256x256x64_w8"),        # first size at which the staged tiles serve a small batch
    (640, 28672, "gemm_fused_staged_256x192x64_w8"),
])
@pytest.mark.parametrize("mode", [wl.BUCKET_SORTED, wl.BUCKET_RUNS])
def test_staged_tile_choice(n_tokens, cols, kernel, mode):
    # a short K keeps the oracle quick: the choice depends on the tile counts (256 CUs); few runs of one adapter and rows without one
    rng = np.random.default_rng(n_tokens)
    ids = np.repeat(rng.integers(-1, 12, size=n_tokens // 9 + 1), 9)[:n_tokens].astype(np.int32)
    w = wl.custom("staged_tiles", 3, [(128, cols)], ["p"], 12, 32, mode, ids, {i: 8 * (1 + i % 4) for i in range(12)})
    sess = Session(w)
    try:
        sess.load(w.resident)
        sess.bucket()
        sess.forward(0)
        assert kernel in B.lora_last_launches(sess.ctx), B.lora_last_launches(sess.ctx)
    finally:
        sess.close()
    run_and_check(w)


def _large_operand(T, K, cols, gated=False, tuning=None):
    """One call without adapters on operands of 4 GiB, compared with the fp32 product at the rows and columns around
    byte 2^32 of x and W, at the ends and at random places."""
    dev = torch.device("cuda:0")
    n = 2 if gated else 1
    cfg = B.make_config([(K, cols)] * n, 1, 8, T, 1)
    nbytes = B.lora_slab_bytes(cfg)
    slab = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    cfg.slab, cfg.slab_bytes = slab.data_ptr(), nbytes
    ctx = B.lora_create(cfg)
    try:
        for key, value in (tuning or {}).items():
            B.lora_set_tuning(ctx, key, value)
        gen = torch.Generator(device=dev).manual_seed(T + cols)
        x = torch.empty((T, K), dtype=torch.bfloat16, device=dev).normal_(generator=gen)
        W = [torch.empty((cols, K), dtype=torch.bfloat16, device=dev).normal_(0.0, 0.02, generator=gen) for _ in range(n)]
        y = torch.empty((T, cols), dtype=torch.bfloat16, device=dev)
        ids = torch.full((T,), -1, dtype=torch.int32, device=dev)
        st = torch.cuda.current_stream().cuda_stream
        seg = B.lora_bucket(ctx, ids.data_ptr(), T, B.LORA_BUCKET_RUNS, st)
        if gated:
            B.lora_layer_forward_glu(ctx, 0, 1, x.data_ptr(), W[0].data_ptr(), W[1].data_ptr(), seg, y.data_ptr(), st)
        else:
            B.lora_layer_forward(ctx, 0, x.data_ptr(), W[0].data_ptr(), seg, y.data_ptr(), st)
        print(f"[gpu-case] T={T} K={K} cols={cols} {B.lora_last_launches(ctx)}", flush=True)
        edge = 2 ** 31 // K
        rng = np.random.default_rng(1)

        def picks(size):
            return sorted({i for i in [0, 1, 2, 3, edge - 1, edge, edge + 1, edge + 2, edge + 3, size - 2, size - 1, *rng.integers(0, size, 40)] if i < size})

        r, c = torch.tensor(picks(T), device=dev), torch.tensor(picks(cols), device=dev)
        ref = [x[r].float() @ m[c].float().t().contiguous() for m in W]
        ref = torch.nn.functional.silu(ref[0]) * ref[1] if gated else ref[0]
        got = y[r][:, c].float()
        assert float((got - ref).abs().max() / ref.abs().max()) <= 5e-3
    finally:
        B.lora_destroy(ctx)


@pytest.mark.parametrize("T", [257, 1100])
@pytest.mark.parametrize("gated", [False, True])
def test_weights_of_4_gib(T, gated):
    _large_operand(T, 16384, 131080, gated)


@pytest.mark.parametrize("tuning", [{}, {B.LORA_TUNE_FUSED_VARIANT: B.FUSED_VARIANTS["256x128x32_w8"]}])
def test_activations_of_4_gib(tuning):
    _large_operand(200003, 16384, 200, tuning=tuning)


def test_weights_of_4_gib_in_an_explicit_split_variant():
    _large_operand(100, 2 ** 21, 1032, tuning={B.LORA_TUNE_SPLIT_VARIANT: B.SPLIT_VARIANTS["256x128x32_w4"]})


@pytest.mark.parametrize("mode,launches", [(B.LORA_INLINE_SHRINK_ON, ["gemm_fused_256x256x64_w8"]),
                                           (B.LORA_INLINE_SHRINK_AUTO, ["shrink", "gemm_fused_staged_256x256x64_w8"])])
def test_shrink_inside_a_wide_launch_of_more_than_256_tokens(mode, launches):
    # 224 tiles of 256 x 256: 32 CUs without a tile
    ids = np.random.default_rng(9).integers(-1, 6, size=400).astype(np.int32)
    w = wl.custom("wide_inline", 9, [(128, 28672)], ["p"], 6, 16, wl.BUCKET_SORTED, ids, {i: 8 * (1 + i % 2) for i in range(6)})
    tuning = {B.LORA_TUNE_INLINE_SHRINK: mode}
    assert _launches(w, tuning) == launches
    run_and_check(w, tuning=tuning)


@pytest.mark.parametrize("mode", [B.LORA_INLINE_SHRINK_OFF, B.LORA_INLINE_SHRINK_ON])
@pytest.mark.parametrize("name", ["32x128x64_w4", "64x128x64_w4", "32x128x64_w4_pair", "64x128x64_w4_pair"])
def test_shrink_inside_the_small_tiles(mode, name):
    tuning = {B.LORA_TUNE_INLINE_SHRINK: mode, B.LORA_TUNE_FUSED_VARIANT: B.FUSED_VARIANTS[name]}
    for n_tokens in (1, 33, 64):
        w = wl.config2(shrink=8, n_tokens=n_tokens)
        inside = mode == B.LORA_INLINE_SHRINK_ON
        assert _launches(w, tuning, B.LORA_PATH_FUSED) == ([] if inside else ["shrink"]) + ["gemm_fused_" + name]
        run_and_check(w, path=B.LORA_PATH_FUSED, tuning=tuning, packed=True)


@pytest.mark.parametrize("mode", [B.LORA_INLINE_SHRINK_OFF, B.LORA_INLINE_SHRINK_ON])
@pytest.mark.parametrize("n_tokens,kernel", [(1, "gemm_fused_32x128x64_w4_pair"), (32, "gemm_fused_32x128x64_w4_pair"),
                                             (33, "gemm_fused_64x128x64_w4_pair"), (64, "gemm_fused_64x128x64_w4_pair"),
                                             (65, "gemm_fused_128x128x64_w4")])
def test_more_small_tiles_than_cus(n_tokens, kernel, mode):
    # 258 column tiles of 128 for 256 CUs, the last one ragged; the 128-row tile leaves no CU for the shrink
    ids = np.random.default_rng(n_tokens).integers(-1, 6, size=n_tokens).astype(np.int32)
    w = wl.custom("pair_tiles", 11, [(320, 33000)], ["p"], 6, 16, wl.BUCKET_SORTED, ids, {i: 8 * (1 + i % 2) for i in range(6)})
    tuning = {B.LORA_TUNE_INLINE_SHRINK: mode}
    inside = mode == B.LORA_INLINE_SHRINK_ON and n_tokens <= 64
    assert _launches(w, tuning) == ([] if inside else ["shrink"]) + [kernel]
    run_and_check(w, tuning=tuning)


@pytest.mark.parametrize("n_tokens,rows", [(1, 32), (31, 32), (32, 32), (33, 64), (63, 64), (64, 64), (65, 128)])
def test_small_batch_tiles_by_name(n_tokens, rows):
    w = wl.config2(shrink=8, n_tokens=n_tokens)
    assert _launches(w, path=B.LORA_PATH_FUSED)[-1] == f"gemm_fused_{rows}x128x64_w4"
    assert _launches(w, path=B.LORA_PATH_SPLITK) == [f"gemm_splitk_shrink_{rows}x128x64_w4", "reduce_expand"]


@pytest.mark.parametrize("value", [24, 29, 32, 1000])
def test_unknown_variants_fall_back(value):
    w = wl.config2(shrink=8, n_tokens=100)
    run_and_check(w, path=B.LORA_PATH_FUSED, tuning={B.LORA_TUNE_FUSED_VARIANT: value})
    run_and_check(w, path=B.LORA_PATH_SPLITK, tuning={B.LORA_TUNE_SPLIT_VARIANT: value})
    assert _launches(w, {B.LORA_TUNE_FUSED_VARIANT: value}, B.LORA_PATH_FUSED)[-1] == "gemm_fused_256x256_w8"
    assert _launches(w, {B.LORA_TUNE_SPLIT_VARIANT: value}, B.LORA_PATH_SPLITK)[0] == "gemm_splitk_shrink_256x128_w8"


@pytest.mark.parametrize("n_tokens", [65, 128])
def test_turned_k_walk_of_the_128_row_tile(n_tokens):
    # K of gate|up 2048: 32 K tiles, 112 column tiles; and a K that does not turn the walk, behind it on the same sizes
    run_and_check(wl.config2(shrink=2, n_tokens=n_tokens), path=B.LORA_PATH_FUSED, packed=True)
    run_and_check(wl.qwen_decode(shrink=2, n_tokens=n_tokens), path=B.LORA_PATH_FUSED, packed=True)


@pytest.mark.parametrize("n_tokens,cols,launches", [
    # two full rounds of 256 x 256 tiles and 8 rows (their split-K pass costs less than 256 x 192 tiles in three rounds)
    (8200, 4096, ["gemm_fused_direct_256x256x64_w4", "gemm_splitk_shrink_256x128x64_w8", "reduce_expand"]),
    # one full round would be followed by 1104 rows, more than the split-K path takes
    (5200, 4096, ["gemm_fused_direct_256x192x64_w4"]),
])
def test_rows_behind_the_full_rounds(n_tokens, cols, launches):
    ids = np.full(n_tokens, -1, dtype=np.int32)
    w = wl.custom("tail", 12, [(4096, cols)], ["p"], 1, 8, wl.BUCKET_RUNS, ids, {0: 8}, resident=[])
    sess = Session(w)
    try:
        sess.bucket()
        y = sess.forward(0).float()
        assert B.lora_last_launches(sess.ctx) == launches
        ref = sess.x[0].float() @ sess.W[0].float().t().contiguous()
        assert float((y - ref).abs().max() / ref.abs().max()) <= 5e-3
    finally:
        sess.close()

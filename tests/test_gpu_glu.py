"""GPU parity of gate and up in one call with their product (lora_layer_forward_glu): silu(gate) * up against the
oracle's float64 definition, on the three kernels that serve it (128-row and 256-row small-batch tiles, the
register-staged prefill tile), with many adapters, without any, and from a pool of pages."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, announce, check_segments, rel_err
from paper_2602_24044_amd import binding as B
from paper_2602_24044_amd import workloads as wl
from paper_2602_24044_amd.runtime import Session, bf16_tensor_to_bits

pytestmark = pytest.mark.gpu


def _gate_up(w):
    return w.proj_names.index("gate"), w.proj_names.index("up")


def _run(w, expect_kernel, n_pages=0, ids=None):
    g, u = _gate_up(w)
    if ids is not None:
        w.token_ids = ids
    announce(f"glu {w.name} T={w.T} proj={w.proj[g]} n_pages={n_pages}")
    sess = Session(w, n_pages=n_pages)
    try:
        sess.load(w.resident)
        sess.bucket(torch.from_numpy(w.token_ids).to(sess.device))
        assert check_segments(sess, w) == 0
        out = sess.forward_glu(g, u)
        torch.cuda.synchronize()
        launches = B.lora_last_launches(sess.ctx)
        h_ref = oracle.gated(w.x[g], w.W[g], w.W[u], w.token_ids, oracle.adapters_of(w, g), oracle.adapters_of(w, u))
        e = rel_err(bf16_tensor_to_bits(out), h_ref)
        announce(f"  launches={launches} rel_err={e:.3e}")
        assert expect_kernel in launches, launches
        assert e <= TOL
        # and the separate projections still come out as before on the same context
        for p in (g, u):
            y = sess.forward(p)
            torch.cuda.synchronize()
            y_ref = oracle.project(w.x[p], w.W[p], w.token_ids, oracle.adapters_of(w, p))
            assert rel_err(bf16_tensor_to_bits(y), y_ref) <= TOL
        assert B.lora_poll_device_flags(sess.ctx) == (B.LORA_OK, 0)
    finally:
        sess.close()


def test_small_batch_tiles():
    _run(wl.config2(shrink=8, n_tokens=100), "gemm_glu_128x128x64_w4")
    _run(wl.config2(shrink=8, n_tokens=300), "gemm_glu_256x128x64_w8")
    _run(wl.config2(shrink=4, n_tokens=777), "gemm_glu_256x128x64_w8")


def test_prefill_tile_and_ragged_sizes():
    _run(wl.config3(shrink=8, n_req=6, len_div=4), "gemm_glu_staged_256x256x64_w8")
    _run(wl.qwen_decode(shrink=8, n_tokens=150), "gemm_glu_256x128x64_w8")          # 18944 / 8 = 2368 columns: ragged last tile


def test_many_adapters_none_and_a_pool_of_pages():
    w = wl.config4(shrink=8, n_tokens=400, n_adapters=96)
    _run(w, "gemm_glu_256x128x64_w8")
    _run(wl.config4(shrink=8, n_tokens=400, n_adapters=96), "gemm_glu_256x128x64_w8",
         n_pages=sum(w.adapters[a].rank // 8 for a in w.resident))
    w = wl.config2(shrink=8, n_tokens=300)
    _run(w, "gemm_glu_256x128x64_w8", ids=np.full(w.T, -1, dtype=np.int32))


def test_argument_errors():
    w = wl.qwen_decode(shrink=8, n_tokens=40)
    sess = Session(w)
    try:
        sess.load(w.resident)
        sess.bucket()
        g, u = _gate_up(w)
        q, k = w.proj_names.index("q"), w.proj_names.index("k")
        out = torch.empty((w.T, w.proj[g][1]), dtype=torch.bfloat16, device=sess.device)
        for pa, pb, status in ((g, g, B.LORA_ERR_INVALID_ARG), (g, 99, B.LORA_ERR_INVALID_ARG), (q, k, B.LORA_ERR_SHAPE)):
            with pytest.raises(B.LoraError) as e:
                B.lora_layer_forward_glu(sess.ctx, pa, pb, sess.x[g].data_ptr(), sess.W[g].data_ptr(), sess.W[u].data_ptr(),
                                         sess.seg, out.data_ptr())
            assert e.value.status == status
        # projections with a bias (q and v of this family have one and the same shape only if kv = hidden; use k, v)
        kk, v = w.proj_names.index("k"), w.proj_names.index("v")
        with pytest.raises(B.LoraError) as e:
            B.lora_layer_forward_glu(sess.ctx, kk, v, sess.x[kk].data_ptr(), sess.W[kk].data_ptr(), sess.W[v].data_ptr(),
                                     sess.seg, out.data_ptr())
        assert e.value.status == B.LORA_ERR_INVALID_ARG
    finally:
        sess.close()


@pytest.mark.parametrize("n_tokens,kernel", [(1, "gemm_glu_64x128x64_w4"), (64, "gemm_glu_64x128x64_w4"), (65, "gemm_glu_128x128x64_w4")])
def test_smallest_batches(n_tokens, kernel):
    _run(wl.config2(shrink=8, n_tokens=n_tokens), kernel)
    _run(wl.qwen_decode(shrink=8, n_tokens=n_tokens), kernel)


def test_gated_tile_of_eight_waves():
    # at least half as many 128 x 128 tiles of both matrices as CUs: 2 x 8192 columns; a short K keeps the oracle quick
    rng = np.random.default_rng(5)
    ids = rng.integers(-1, 6, size=101).astype(np.int32)
    w = wl.custom("glu_wide", 5, [(128, 8200), (128, 8200)], ["gate", "up"], 6, 16, wl.BUCKET_SORTED, ids, {i: 8 * (1 + i % 2) for i in range(6)})
    _run(w, "gemm_glu_128x128x64_w8")
    # more 64-row tiles than CUs: two workgroups on a CU
    w = wl.custom("glu_wider", 6, [(128, 16648), (128, 16648)], ["gate", "up"], 6, 16, wl.BUCKET_SORTED, ids[:40], {i: 8 * (1 + i % 2) for i in range(6)})
    _run(w, "gemm_glu_64x128x64_w4_pair")


def test_staged_gated_tile_below_1025_tokens():
    rng = np.random.default_rng(7)
    ids = np.repeat(rng.integers(-1, 6, size=30), 10)[:261].astype(np.int32)
    w = wl.custom("glu_staged", 7, [(64, 14336), (64, 14336)], ["gate", "up"], 6, 16, wl.BUCKET_SORTED, ids, {i: 8 * (1 + i % 2) for i in range(6)})
    _run(w, "gemm_glu_staged_256x256x64_w8")


@pytest.mark.parametrize("n_tokens,cols,kernel", [(520, 14336, "gemm_glu_256x128x64_w8"),        # 3 rounds of 256 x 128 tiles against 2
                                                  (777, 14336, "gemm_glu_staged_256x256x64_w8"), # 4 against 2
                                                  (300, 18944, "gemm_glu_256x128x64_w8"),        # 3 against 2
                                                  (850, 18944, "gemm_glu_256x128x64_w8"),        # 5 against 3
                                                  (1025, 18944, "gemm_glu_staged_256x256x64_w8")])
def test_gated_tile_by_rounds(n_tokens, cols, kernel):
    rng = np.random.default_rng(n_tokens)
    ids = np.repeat(rng.integers(-1, 6, size=n_tokens // 10 + 1), 10)[:n_tokens].astype(np.int32)
    w = wl.custom("glu_rounds", 8, [(64, cols), (64, cols)], ["gate", "up"], 6, 16, wl.BUCKET_SORTED, ids, {i: 8 * (1 + i % 2) for i in range(6)})
    _run(w, kernel)


@pytest.mark.parametrize("mode", [B.LORA_INLINE_SHRINK_OFF, B.LORA_INLINE_SHRINK_ON])
@pytest.mark.parametrize("n_tokens,kernel", [(1, "gemm_glu_64x128x64_w4"), (64, "gemm_glu_64x128x64_w4"), (65, "gemm_glu_128x128x64_w4"),
                                             (129, "gemm_glu_256x128x64_w8")])
def test_gated_shrink_inside_and_outside_the_launch(n_tokens, kernel, mode):
    # an adapter of the largest rank per token over a short K: the tiles arrive first.  Every second launch has NaN for x, so
    # a tile that does not wait for its own launch's shrink results shows it
    n_ad = min(n_tokens, 64)
    ids = (np.arange(n_tokens) % n_ad).astype(np.int32)
    w = wl.custom("glu_late_shrink", 43 + n_tokens, [(512, 1792), (512, 1792)], ["gate", "up"], n_ad, 64, wl.BUCKET_SORTED, ids,
                  {i: 64 for i in range(n_ad)})
    announce(f"glu wait T={n_tokens} mode={mode} {kernel}")
    sess = Session(w)
    try:
        B.lora_set_tuning(sess.ctx, B.LORA_TUNE_INLINE_SHRINK, mode)
        sess.load(w.resident)
        sess.bucket()
        x_ok, x_nan = sess.x, [torch.full_like(t, float("nan")) for t in sess.x]
        outs = []
        for rep in range(20):
            sess.x = x_nan if rep % 2 == 0 else x_ok
            y = sess.forward_glu(0, 1)
            assert B.lora_last_launches(sess.ctx) == (["shrink"] if mode == B.LORA_INLINE_SHRINK_OFF else []) + [kernel]
            if rep % 2:
                outs.append(y)
        torch.cuda.synchronize()
        h_ref = oracle.gated(w.x[0], w.W[0], w.W[1], w.token_ids, oracle.adapters_of(w, 0), oracle.adapters_of(w, 1))
        assert rel_err(bf16_tensor_to_bits(outs[0]), h_ref) <= TOL
        assert all(torch.equal(y, outs[0]) for y in outs)
        assert B.lora_poll_device_flags(sess.ctx) == (B.LORA_OK, 0)
    finally:
        sess.close()

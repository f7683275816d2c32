"""GPU parity of moe_expert_ffn (SwiGLU experts weighted by gating
probabilities, Section 2) against the fp64 oracle: relative L2 <= 1e-2."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-2


def _gpu_ffn(cfg, layer, idx, w, x_store, n_shared=0):
    """moe_expert_ffn on seeded blobs of the row's valid experts."""
    import torch
    from gpuhelp import DEV, blob_dev, i32, ptr_array, storage_dtype, to_dev
    from paper_2606_15453_amd import stmoe as S
    B, K = idx.shape
    sel = sorted(e for e in set(idx.ravel().tolist()) if 0 <= e < cfg.E)
    blobs = {e: blob_dev(cfg, layer, e) for e in sel}
    ptrs = [blobs[e].data_ptr() if e in blobs else 0 for e in range(cfg.E)]
    shared = [blob_dev(cfg, layer, s, shared=True) for s in range(n_shared)]
    y = torch.full((B, cfg.H), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.zeros(S.ffn_workspace_bytes(B, K, cfg.E, cfg.H, cfg.I, n_shared, storage_dtype(cfg)),
                     dtype=torch.uint8, device=DEV)
    S.expert_ffn(to_dev(x_store), i32(idx), torch.from_numpy(w.astype(np.float32)).to(DEV), cfg.H,
                 cfg.I, cfg.E, storage_dtype(cfg), ptr_array(ptrs), y, ws,
                 shared_ptrs=ptr_array([s.data_ptr() for s in shared]) if n_shared else None,
                 n_shared=n_shared)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def _run_ffn(cfg, layer, idx, w, x_store, n_shared=0):
    from gpuhelp import expert_f64, rel_l2
    from oracle.stmoe_oracle import decode_storage, moe_ffn
    got = _gpu_ffn(cfg, layer, idx, w, x_store, n_shared)
    ref = moe_ffn(decode_storage(x_store), idx, w, lambda e: expert_f64(cfg, layer, e),
                  shared=[expert_f64(cfg, layer, s, shared=True) for s in range(n_shared)])
    return got, ref, rel_l2(got, ref)


def _inputs(cfg, B, K, seed, distinct_rows=True):
    from paper_2606_15453_amd import workload as W
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.choice(cfg.E, K, replace=False) for _ in range(B)]).astype(np.int32)
    w = rng.dirichlet(np.ones(cfg.E), size=B)[:, :K].astype(np.float32) + 0.05
    x = rng.normal(0, 1, (B, cfg.H))
    return idx, w, W.to_storage(cfg, x)


@pytest.mark.parametrize("name,B", [("tiny", 1), ("qwen30b", 1), ("dsv2lite", 1), ("qwen30b", 3), ("qwen30b-b8", 8),
                                    ("qwen30b-b8", 12), ("dsv2lite", 4), ("dsv2lite", 9),
                                    ("qwen235b", 16), ("qwen235b", 9), ("qwen235b", 2), ("qwen235b", 4),
                                    ("mixtral", 4), ("mixtral", 8)])
def test_ffn_parity(name, B):
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS[name].scaled(B=B)
    idx, w, x = _inputs(cfg, B, cfg.K, seed=B + len(name))
    got, ref, err = _run_ffn(cfg, 1, idx, w, x, n_shared=cfg.n_shared)
    print(f"{name} B={B}: rel L2 {err:.3e}")
    assert np.isfinite(got).all()
    assert err <= TOL


@pytest.mark.parametrize("H,I", [(4096, 1536), (4096, 1472), (4032, 1536)])
def test_ffn_mfma_tiled_shapes(H, I):
    """Batch 16 over 128 experts takes the tiled MFMA gate/up: through LDS with
    two 16-row tiles per wave (H % 128 == 0, I % 128 == 0), with one tile
    (I % 128 != 0), and the direct-load kernel (H % 128 != 0)."""
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["qwen235b"].scaled(H=H, I=I, B=16)
    idx, w, x = _inputs(cfg, 16, cfg.K, seed=H + I)
    got, ref, err = _run_ffn(cfg, 2, idx, w, x)
    print(f"H={H} I={I}: rel L2 {err:.3e}")
    assert np.isfinite(got).all()
    assert err <= TOL


def test_ffn_parity_mixtral_shape():
    """Full Mixtral-8x7B expert shape (H 4096, I 14336), batch 1, top-2."""
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["mixtral"]
    idx, w, x = _inputs(cfg, 1, 2, seed=5)
    got, ref, err = _run_ffn(cfg, 0, idx, w, x)
    print(f"mixtral: rel L2 {err:.3e}")
    assert err <= TOL


def test_ffn_shared_tokens_overlap():
    """Several rows selecting the same experts: each expert is read once and
    its tokens are grouped; ragged sizes (H and I not multiples of 64 chunks)."""
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["qwen30b"].scaled(H=264, I=40, E=10, K=3, B=6)
    idx = np.array([[0, 1, 2], [2, 1, 0], [9, 0, 4], [4, 9, 1], [3, 5, 7], [0, 2, 1]], np.int32)
    w = np.random.default_rng(2).random((6, 3)).astype(np.float32)
    x = W.to_storage(cfg, np.random.default_rng(3).normal(0, 1, (6, cfg.H)))
    got, ref, err = _run_ffn(cfg, 0, idx, w, x)
    assert err <= TOL


@pytest.mark.parametrize("B", [8, 11])
def test_ffn_batch8_fallback_shapes(B):
    """Batch >= 8 with H, I not multiples of 64 runs the GEMV kernels."""
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["qwen30b"].scaled(H=264, I=40, E=12, K=3, B=B)
    idx, w, x = _inputs(cfg, B, 3, seed=B)
    got, ref, err = _run_ffn(cfg, 0, idx, w, x)
    assert err <= TOL


def test_ffn_repeated_calls_reuse_workspace():
    """Completion tickets in the workspace are reset by every call."""
    import torch
    from gpuhelp import DEV, blob_dev, expert_f64, i32, ptr_array, rel_l2, storage_dtype, to_dev
    from oracle.stmoe_oracle import decode_storage, moe_ffn
    from paper_2606_15453_amd import stmoe as S
    from paper_2606_15453_amd import workload as W
    for name, B in (("qwen30b", 1), ("qwen235b", 16)):
        cfg = W.CONFIGS[name].scaled(B=B, E=24)
        blobs = [blob_dev(cfg, 0, e) for e in range(cfg.E)]
        ptrs = ptr_array([b.data_ptr() for b in blobs])
        ws = torch.zeros(S.ffn_workspace_bytes(B, cfg.K, cfg.E, cfg.H, cfg.I, 0, storage_dtype(cfg)),
                         dtype=torch.uint8, device=DEV)
        y = torch.empty((B, cfg.H), dtype=torch.float32, device=DEV)
        for rep in range(3):
            idx, w, x = _inputs(cfg, B, cfg.K, seed=100 + rep)
            S.expert_ffn(to_dev(x), i32(idx), torch.from_numpy(w).to(DEV), cfg.H, cfg.I, cfg.E,
                         storage_dtype(cfg), ptrs, y, ws)
            ref = moe_ffn(decode_storage(x), idx, w, lambda e: expert_f64(cfg, 0, e))
            assert rel_l2(y.cpu().numpy(), ref) <= TOL


def test_ffn_zero_input_and_linearity():
    import torch
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["qwen30b"].scaled(B=2)
    idx, w, x = _inputs(cfg, 2, cfg.K, seed=9)
    got0, _, _ = _run_ffn(cfg, 0, idx, w, np.zeros_like(x))
    assert np.all(got0 == 0)
    g1, _, _ = _run_ffn(cfg, 0, idx, w, x)
    g2, _, _ = _run_ffn(cfg, 0, idx, 2 * w, x)
    assert np.allclose(g2, 2 * g1, rtol=1e-5, atol=1e-7)


def test_ffn_deterministic():
    from paper_2606_15453_amd import workload as W
    cfg = W.CONFIGS["qwen30b"].scaled(B=4)
    idx, w, x = _inputs(cfg, 4, cfg.K, seed=11)
    a, _, _ = _run_ffn(cfg, 2, idx, w, x)
    b, _, _ = _run_ffn(cfg, 2, idx, w, x)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("name,row", [("qwen30b", [5, 9, 5, -1, 17, 9, 3, 130]), ("tiny", [3, 3]),
                                      ("dsv2lite", [7, 200, 7, 1, 63, -5])])
def test_ffn_repeated_and_out_of_range_entries(name, row):
    """A selection row that repeats an expert or holds an index outside
    [0, E): out-of-range entries are ignored and a repeated expert counts once,
    with the weight of its first entry (batch 1 takes the register slot
    lookup; batch 2 repeats the row and takes the slot plan).  Checked against
    the oracle on the row's distinct valid entries."""
    from paper_2606_15453_amd import workload as W
    base = W.CONFIGS[name]
    K = len(row)
    for B in (1, 2):
        cfg = base.scaled(B=B, K=K, E=max(base.E, K))
        rng = np.random.default_rng(K + B)
        idx = np.array([row] * B, dtype=np.int32)
        w = (rng.random((B, K)) + 0.1).astype(np.float32)
        x = W.to_storage(cfg, rng.normal(0, 1, (B, cfg.H)))
        keep = [k for k in range(K) if 0 <= row[k] < cfg.E and row[k] not in row[:k]]
        got = _gpu_ffn(cfg, 1, idx, w, x, n_shared=cfg.n_shared)
        _, ref, _ = _run_ffn(cfg, 1, idx[:, keep].copy(), w[:, keep].copy(), x, n_shared=cfg.n_shared)
        from gpuhelp import rel_l2
        err = rel_l2(got, ref)
        print(f"{name} B={B} row {row}: rel L2 against the oracle on {len(keep)} entries {err:.3e}")
        assert np.isfinite(got).all() and err <= TOL



@pytest.mark.parametrize("B,K,E,H,I,n_shared,dtype", [
    (2, 1, 3, 8, 8, 0, "bf16"),          # one chunk per row: the columns' remainder is all there is
    (3, 2, 60, 136, 24, 1, "bf16"),      # one full step and a remainder, rows not a multiple of a wave's
    (4, 6, 64, 2048, 1408, 2, "bf16"),   # split columns, no remainder, two row quads per down wave
    (5, 3, 10, 1032, 40, 0, "f32"),      # fp32, two token groups, remainder of two chunks
    (6, 4, 60, 2056, 1000, 1, "bf16"),   # 257 pairs of row quads: one quad per down wave
    (8, 8, 128, 2048, 768, 0, "bf16"),   # the largest batch of two token groups
    (8, 8, 8, 256, 64, 0, "f32"),        # every token in every slot: both token groups full
    (5, 3, 20, 576, 192, 1, "bf16"),     # rows of whole cache lines that end inside a 256-byte step
    (4, 2, 12, 584, 200, 1, "f32"),      # rows that share cache lines
    (9, 1, 1, 72, 104, 0, "bf16"),       # one expert serves nine tokens: four token groups
    (14, 1, 26, 704, 2192, 0, "bf16"),   # batch beyond 8 with sizes the 16-row tiles do not take
    (16, 2, 5, 64, 8, 8, "f32"),         # the largest batch, eight shared experts
    (16, 16, 256, 128, 64, 0, "bf16"),   # the largest K and E: 16-row down after 4-row gate/up
    (16, 4, 8, 128, 64, 0, "bf16"),      # many tokens per slot: 16-row gate/up
    (8, 5, 18, 1032, 264, 1, "f32"),     # short rows in few workgroups: split columns, remainder, two token groups
    (8, 5, 6, 4096, 128, 1, "bf16"),     # batch 8, many tokens per slot, long rows: 16-row tiles
    (8, 8, 70, 256, 768, 0, "bf16"),     # batch 8, short outputs of many slots: 16-row tiles
    (3, 3, 20, 1416, 1192, 1, "bf16"),   # ... in many: not split, 11 steps and a remainder
])
def test_ffn_tile_edges(B, K, E, H, I, n_shared, dtype):
    """The 4-row tile kernels at the edges of their tiles, token groups and
    splits.  fp32: the oracle's fp64 result within 1e-5 (sums of at most
    2064 products, errors of a few fp32 roundings, 6e-8 each, per chained sum
    of at most 64); bf16: weights and inputs are exact, activations rounded to
    bf16 (2^-9 each)."""
    from paper_2606_15453_amd import workload as W
    base = W.CONFIGS["tiny" if dtype == "f32" else "qwen30b"]
    cfg = base.scaled(H=H, I=I, E=E, K=K, B=B, dtype=dtype)
    idx, w, x = _inputs(cfg, B, K, seed=B * 100 + H + I)
    got, ref, err = _run_ffn(cfg, 1, idx, w, x, n_shared=n_shared)
    print(f"B={B} K={K} E={E} H={H} I={I} +{n_shared} {dtype}: rel L2 {err:.3e}")
    assert np.isfinite(got).all()
    assert err <= (1e-5 if dtype == "f32" else TOL)


@pytest.mark.parametrize("B,dtype,H,I", [(3, "bf16", 264, 72), (6, "f32", 264, 72), (7, "bf16", 256, 128)])
def test_ffn_non_finite_weights_stay_with_their_tokens(B, dtype, H, I):
    """An expert whose W_down holds an infinity (or whose W_gate holds a NaN)
    changes only the rows routed to it, also where its tile serves other rows
    beside them."""
    import torch
    from gpuhelp import DEV, blob_dev, i32, ptr_array, storage_dtype, to_dev
    from paper_2606_15453_amd import stmoe as S
    from paper_2606_15453_amd import workload as W
    base = W.CONFIGS["tiny" if dtype == "f32" else "qwen30b"]
    cfg = base.scaled(H=H, I=I, E=6, K=2, B=B, dtype=dtype)
    _, w, x = _inputs(cfg, B, 2, seed=3)
    idx = np.array([[b % 3, 3 + b % 3] for b in range(B)], np.int32)      # expert 0: rows 0, 3, 6
    ys = []
    for bad in (False, True):
        blobs = [blob_dev(cfg, 0, e) for e in range(cfg.E)]
        if bad:
            blobs[0][2 * H * I:].fill_(float("inf"))
            blobs[4][:H].fill_(float("nan"))                              # expert 4: rows 1, 4
        y = torch.empty((B, H), dtype=torch.float32, device=DEV)
        ws = torch.zeros(S.ffn_workspace_bytes(B, 2, 6, H, I, 0, storage_dtype(cfg)), dtype=torch.uint8, device=DEV)
        S.expert_ffn(to_dev(x), i32(idx), torch.from_numpy(w).to(DEV), H, I, 6, storage_dtype(cfg),
                     ptr_array([b.data_ptr() for b in blobs]), y, ws)
        ys.append(y.cpu().numpy())
    for b in range(B):
        if b % 3 == 2:
            assert np.array_equal(ys[0][b], ys[1][b]), b
        else:
            assert not np.isfinite(ys[1][b]).any(), b


def _ffn_launches(B, K, E, H, I, n_shared, dtype):
    import torch
    from gpuhelp import DEV, graph_launches, ptr_array
    from paper_2606_15453_amd import stmoe as S
    dt, sdt = (torch.bfloat16, S.BF16) if dtype == "bf16" else (torch.float32, S.F32)
    x = torch.zeros((B, H), dtype=dt, device=DEV)
    idx, w = torch.zeros((B, K), dtype=torch.int32, device=DEV), torch.zeros((B, K), device=DEV)
    y = torch.zeros((B, H), device=DEV)
    ws = torch.zeros(S.ffn_workspace_bytes(B, K, E, H, I, n_shared, sdt), dtype=torch.uint8, device=DEV)
    table, st = ptr_array([x.data_ptr()] * (E + n_shared)), torch.cuda.Stream()      # captured, not run
    shared = table if n_shared else None
    return graph_launches(lambda: S.expert_ffn(x, idx, w, H, I, E, sdt, table, y, ws, shared_ptrs=shared,
                                               n_shared=n_shared, stream=st), st)


@pytest.mark.parametrize("B,K,E,H,I,n_shared,dtype,rows", [
    (8, 8, 32, 1024, 1024, 0, "bf16", 16), (8, 4, 43, 1024, 1920, 0, "bf16", 16),
    (3, 6, 16, 1408, 4096, 1, "bf16", 16), (3, 6, 16, 1536, 1024, 1, "bf16", 4),
    (5, 4, 157, 640, 1152, 0, "f32", 16), (4, 6, 64, 2048, 1408, 2, "bf16", 4), (8, 5, 18, 1280, 400, 2, "bf16", 4),
    (8, 4, 8, 256, 64, 0, "bf16", 16),
])
def test_gate_up_tile_splits(B, K, E, H, I, n_shared, dtype, rows):
    """Rows per gate/up workgroup of the 4-row tiles: columns split over its
    waves (4 rows) for long rows, and for shorter ones in few workgroups."""
    slots = min(B * K, E) + n_shared
    up = _ffn_launches(B, K, E, H, I, n_shared, dtype)[0]
    assert up == (-(-I // rows) * slots + 1, 256)        # one more publishes the plan


@pytest.mark.parametrize("K,E,H,I,n_shared,rows16", [
    (4, 8, 4096, 1024, 0, True), (8, 8, 4096, 14336, 0, True), (4, 16, 4096, 1536, 1, True), (8, 12, 2048, 768, 0, True),
    (2, 8, 4096, 14336, 0, False), (4, 8, 2048, 2048, 0, False), (6, 64, 2048, 1408, 2, False),
    (8, 8, 4032, 1024, 0, False),                             # rows that the 16-row kernels don't stage
    (6, 16, 1536, 3072, 0, True), (6, 32, 1664, 3328, 0, False), (6, 8, 1024, 4096, 0, False), (3, 11, 3968, 7168, 0, False),
    (8, 97, 256, 768, 0, True), (8, 128, 256, 512, 0, False), (8, 64, 384, 1024, 0, True), (8, 64, 512, 1024, 0, False),
])
def test_batch8_tiles(K, E, H, I, n_shared, rows16):
    """Batch 8 takes 16-row tiles (workgroups of four waves throughout) where
    slots serve many tokens or short outputs sum many slots, else 4-row tiles
    (down: eight waves or sixteen)."""
    down = _ffn_launches(8, K, E, H, I, n_shared, "bf16")[1]
    assert down[1] == 256 if rows16 else down[1] >= 512


@pytest.mark.parametrize("K,E,H,I,n_shared,dtype,tile", [
    (1, 9, 416, 1176, 0, "bf16", False), (2, 9, 416, 1176, 0, "bf16", True), (1, 24, 1280, 1280, 1, "bf16", True),
    (6, 23, 1096, 656, 0, "f32", False), (7, 14, 2560, 1280, 0, "f32", False), (1, 31, 888, 2296, 2, "f32", True),
    (4, 60, 2056, 1000, 1, "f32", True), (4, 12, 4096, 1024, 0, "f32", False),
])
def test_batch2_kernels(K, E, H, I, n_shared, dtype, tile):
    """Batch 2: GEMV kernels (the down launch in workgroups of four waves) or
    4-row tiles, and both against the 64-bit oracle."""
    from paper_2606_15453_amd import workload as W
    down = _ffn_launches(2, K, E, H, I, n_shared, dtype)[1]
    assert (down[1] > 256) == tile
    cfg = W.CONFIGS["tiny" if dtype == "f32" else "qwen30b"].scaled(H=H, I=I, E=E, K=K, B=2, dtype=dtype)
    idx, w, x = _inputs(cfg, 2, K, seed=H + I)
    got, ref, err = _run_ffn(cfg, 1, idx, w, x, n_shared=n_shared)
    # fp32: a few roundings of 6e-8 per chained sum of at most 80; bf16: activations rounded (2^-9 each)
    assert np.isfinite(got).all() and err <= (1e-5 if dtype == "f32" else TOL)


@pytest.mark.parametrize("B,K,E,H,I,tile", [
    (9, 1, 8, 2048, 2048, False), (16, 2, 37, 2048, 1152, True), (14, 2, 18, 1664, 896, False), (15, 1, 12, 1408, 1152, True),
    (11, 5, 132, 640, 1536, False), (16, 3, 140, 256, 512, False), (10, 6, 80, 2048, 64, True), (16, 2, 16, 2240, 128, True),
])
def test_gate_up_tiles_beyond_batch_8(B, K, E, H, I, tile):
    """Gate/up beyond batch 8 on 4-row tiles (workgroups of 16 rows, and one
    that publishes the plan) or on 16-row ones, and the result on both."""
    from paper_2606_15453_amd import workload as W
    up = _ffn_launches(B, K, E, H, I, 0, "bf16")[0]
    assert (up[0] == -(-I // 16) * min(B * K, E) + 1) == tile
    if H * I * E < 1 << 27:
        cfg = W.CONFIGS["qwen30b"].scaled(H=H, I=I, E=E, K=K, B=B)
        idx, w, x = _inputs(cfg, B, K, seed=H + I)
        got, ref, err = _run_ffn(cfg, 1, idx, w, x)
        assert np.isfinite(got).all() and err <= TOL

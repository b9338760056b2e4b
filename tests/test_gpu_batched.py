"""The batched products (k_gemm_wide) at the edges of their tiles, k steps and K
parts: a one-layer bf16 decoder whose widths leave remainders everywhere
(d = 4128: 129 k tiles, so steps, parts and folds end in half steps; ffn = 2880;
vocab = 16048: 1003 column tiles).  By row count (256 CUs) the products take every
tile shape, unsplit and split, with ragged rows and columns (folded parts: the
prefill passes below):
  LM head (STORE)    128 x 128 in 8 parts (17 rows), 192 x 256 in 4 and 3 (130, 520),
                     128 x 256 (300), 192 x 256 (700, 1500, 2100) and 256 x 256
                     (2500, 3000) unsplit
  gate/up (SWIGLU)   128 x 128 up to 520 rows, 128 x 256 (700), 192 x 256 (1500,
                     2100, 3000), 256 x 256 (2500)
  O (RESID)          128 x 128 unsplit up to 1500 rows, 192 x 256 (2100, 2500), 256 x
                     256 (3000)
  down (RESID)       split 128 x 128, 128 x 256 and 256 x 256 (17, 130, 700), unsplit
                     128 x 256, 192 x 256, 256 x 256 (1500, 2100, 3000)
  q/k/v (STORE)      split 128 x 128 up to 700 rows, split 128 x 256 above
Sampled rows against the float64 oracle at the bf16 tolerance of the other tests (2e-2:
activations are rounded to bf16 once per product, 2^-9 relative each)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import model as M
from tests.gpu_helpers import check_rows, fill_layer, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 2e-2
CFG = dataclasses.replace(W.config("small_bf16"), name="edges_bf16", L=1, d=4128, hq=2, hkv=1,
                          ffn=2880, vocab=16048)
ROWS = [17, 130, 300, 520, 700, 1500, 2100, 2500, 3000]


@pytest.fixture(scope="module")
def edges():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd.engine import DeviceModel
    print("\n[setup] edges_bf16", flush=True)
    w = W.generate_weights(CFG, seed=0)
    dm = DeviceModel(CFG, n_max=320, gamma_max=4, m_rounds=5, cap_max=80,
                     prefill_chunk=64).upload_all(w)
    yield dm, M.Model(CFG, w)
    dm.close()


def _sample(R):
    return sorted({0, 15, 16, 127, 128, 191, 192, 255, 256, R // 2, R - 2, R - 1} & set(range(R)))


@pytest.mark.parametrize("R", ROWS)
def test_sublayers(edges, R):
    dm, model = edges
    n = 90
    cache = fill_layer(CFG, dm, 0, n, 320)
    x = W.synthetic_rows(R, CFG.d, seed=4, std=0.5, index=800 + R)
    pos = (np.arange(R) % n).astype(np.int32)
    s = _sample(R)
    for i in (1, 2):
        out = torch.empty(R, CFG.d, device="cuda")
        dm.sublayer_apply(i, torch.from_numpy(x).cuda(), pos, mode=1, out=out)
        got = out.cpu().numpy()
        ref = M.sublayer(model, i, x[s].astype(np.float64), pos[s], cache, mode="own")
        check_rows(got[s], x[s], ref, TOL, ("edges", R, i))
        x = got


@pytest.mark.parametrize("R", ROWS)
def test_sublayers_on_rows_at_any_float_address(edges, R):
    """Rows in and out at addresses that are multiples of 4 bytes only: the bits of
    aligned rows, whether the products are split, folded or neither."""
    dm, _ = edges
    n = 90
    fill_layer(CFG, dm, 0, n, 320)
    x = torch.from_numpy(W.synthetic_rows(R, CFG.d, seed=4, std=0.5, index=800 + R)).cuda()
    pos = (np.arange(R) % n).astype(np.int32)
    at = lambda s: torch.full((R * CFG.d + 8,), 7.0, device="cuda")[s:s + R * CFG.d].view(R, -1)
    for i in (1, 2):
        out, x1, out1 = torch.empty_like(x), at(1), at(3)
        x1.copy_(x)
        dm.sublayer_apply(i, x, pos, mode=1, out=out)
        dm.sublayer_apply(i, x1, pos, mode=1, out=out1)
        assert torch.equal(out, out1)
        whole = torch.as_strided(out1, (R * CFG.d + 8,), (1,), 0)
        assert bool((whole[:3] == 7).all() and (whole[3 + R * CFG.d:] == 7).all())


@pytest.mark.parametrize("R", ROWS)
def test_head(edges, R):
    dm, model = edges
    x = torch.from_numpy(W.synthetic_rows(R, CFG.d, seed=4, std=0.5, index=900 + R)).cuda()
    logits, am, top1 = dm.head_rows(x)
    s = _sample(R)
    lg0, _, _ = M.head(model, x.cpu().numpy()[s].astype(np.float64))
    assert rel_err(logits.cpu().numpy()[s], lg0) < TOL
    assert torch.equal(am.long(), logits.argmax(-1))
    # logits at an address that is a multiple of 4 bytes only: the same bits
    from paper_2602_20217_amd import _lib as K
    flat = torch.full((R * CFG.vocab + 8,), 7.0, device="cuda")
    K.ks_head_rows(dm.ctx, x.data_ptr(), R, flat.data_ptr() + 4, am.data_ptr(), top1.data_ptr())
    assert torch.equal(flat[1:1 + R * CFG.vocab].view(R, -1), logits)
    assert bool((flat[0] == 7) & (flat[1 + R * CFG.vocab:] == 7).all())


def test_prefill_passes_keep_the_bits_of_single_chunks(edges):
    """A prefill pass holds as many whole chunks as the row buffers do: 1100
    tokens in chunks of 64 run as one pass of 1088 rows (down projection: 8 parts
    folded in one workgroup, several ending between the k tiles of a step) and a
    ragged chunk; limits that leave room for one chunk run them one by one.  Same
    caches, same token."""
    from paper_2602_20217_amd.engine import DeviceModel
    n = 1100
    cfg = dataclasses.replace(CFG, L=2)
    w = W.generate_weights(cfg, seed=0)
    prompt = W.prompt_ids(cfg.vocab, n)
    runs = []
    for lim in (dict(gamma_max=4, m_rounds=5, cap_max=64), dict(gamma_max=0, m_rounds=1, cap_max=1)):
        dm = DeviceModel(cfg, n_max=n + 20, prefill_chunk=64, **lim).upload_all(w)
        first = dm.prefill(prompt)
        runs.append((first, [t[:, :n].clone() for l in range(2) for t in dm.kv_layer(l)]))
        dm.close()
    assert runs[0][0] == runs[1][0]
    for a, b in zip(runs[0][1], runs[1][1]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("name", ["bf16", "f32"])
def test_prefill_passes_keep_the_history(name):
    """The history rows that a prefill leaves: 1036 tokens in chunks of 128 as one
    pass of 1024 rows and a ragged chunk of 12, against one chunk at a time (limits
    that leave room for no more).  In the bf16 pass q/k/v and O fold 8 parts in one
    workgroup that single chunks split over eight.  Of the 25 history rows 13 come from the pass and 12
    from the ragged chunk.  A selection reads them all: same record, same caches."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd import engine as E
    cfg = (dataclasses.replace(CFG, L=2, hq=16, hkv=8) if name == "bf16" else
           dataclasses.replace(W.config("tiny"), L=2))
    w = W.generate_weights(cfg, seed=0)
    n = 1036
    prompt = W.prompt_ids(cfg.vocab, n)
    params = E.select_params((1.0, 0.0, 1.0), "paper_min", 0, tau=0.0, D=4)  # C = 4
    runs = []
    for cap_max in (64, 4):
        dm = E.DeviceModel(cfg, n_max=n + 20, gamma_max=4, m_rounds=5, cap_max=cap_max,
                           prefill_chunk=128).upload_all(w)
        first = dm.prefill(prompt)
        sel, rec = dm.select(params, debug_cells=3)
        assert sel.C == 4 and sel.n_rows == 25
        runs.append((first, rec, [t[:, :n].clone() for l in range(2) for t in dm.kv_layer(l)]))
        dm.close()
    assert runs[0][0] == runs[1][0]
    for k, v in runs[0][1].items():
        assert np.array_equal(v, runs[1][1][k], equal_nan=v.dtype.kind == "f"), k
    for a, b in zip(runs[0][2], runs[1][2]):
        assert torch.equal(a, b)


@pytest.fixture(scope="module")
def long_ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd.engine import DeviceModel
    cfg = dataclasses.replace(W.config("small_qwen_bf16"), L=1)
    w = W.generate_weights(cfg, seed=0)
    dm = DeviceModel(cfg, n_max=6400, gamma_max=4, m_rounds=5, cap_max=128,
                     prefill_chunk=64).upload_all(w)
    yield cfg, dm, M.Model(cfg, w)
    dm.close()


# 17, 33 and 130 rows x 4 heads: the last workgroup of 64 query vectors holds 4, 4
# and 8 (one column block per wave); 1270 rows at 6200 positions: 40 x 2 x 7
# workgroups of 128 vectors, the last one 88 full (two blocks per wave)
@pytest.mark.parametrize("R,n", [(R, n) for R in (17, 33, 130) for n in (1, 63, 65, 1024, 2049)] +
                         [(1270, 6200)])
def test_batched_attention_edges(long_ctx, R, n):
    """Lengths at the edges of a 64-key tile and of a 1024-position split; row
    lengths differ (position 0 rows see only their own key); keys past the
    cached ones are NaN and must not be read into a result."""
    cfg, dm, model = long_ctx
    cache = fill_layer(cfg, dm, 0, n, 6400)
    for t in dm.kv_layer(0):
        t[:, n:] = float("nan")
    pos = (n - np.arange(R) % min(n + 1, 70)).astype(np.int32)
    x = W.synthetic_rows(R, cfg.d, seed=4, std=0.5, index=40 + R)
    out = torch.empty(R, cfg.d, device="cuda")
    dm.sublayer_apply(1, torch.from_numpy(x).cuda(), pos, mode=1, out=out)
    s = np.arange(R) if R < 1000 else np.r_[0:40, 600:640, R - 40:R]
    ref = M.sublayer(model, 1, x[s].astype(np.float64), pos[s], cache, mode="own")
    check_rows(out.cpu().numpy()[s], x[s], ref, TOL, ("attention", R, n))


@pytest.mark.parametrize("shift", [0, 1])
def test_f32_products_edges(shift):
    """float32 products with fewer k groups than waves (d = 96: 6 groups for 8
    waves), a ragged last row tile and (shift 1) weights that are only 4-byte
    aligned; rows of one launch equal the same rows alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd.engine import DeviceModel
    cfg = dataclasses.replace(W.config("tiny"), name="edges_f32", L=1, d=96, hq=2, hkv=1, ffn=160,
                              vocab=1040)
    w = W.generate_weights(cfg, seed=0)
    dm = DeviceModel(cfg, n_max=64, gamma_max=4, m_rounds=5, cap_max=64, prefill_chunk=16)
    for k in ("wqkv", "wo", "w_gate_up", "w_down"):
        t = dm.w[k][0]
        dm.w[k][0] = torch.empty(t.numel() + shift, device="cuda")[shift:].view(t.shape)
    t = dm.w["lm_head"]
    dm.w["lm_head"] = torch.empty(t.numel() + shift, device="cuda")[shift:].view(t.shape)
    dm.upload_all(w)
    model = M.Model(cfg, w)
    R, n = 21, 10
    cache = fill_layer(cfg, dm, 0, n, 64)
    x = W.synthetic_rows(R, cfg.d, seed=4, std=0.5, index=7)
    pos = (np.arange(R) % n).astype(np.int32)
    for i in (1, 2):
        out, one = torch.empty(R, cfg.d, device="cuda"), torch.empty(1, cfg.d, device="cuda")
        xd = torch.from_numpy(x).cuda()
        dm.sublayer_apply(i, xd, pos, mode=1, out=out)
        ref = M.sublayer(model, i, x.astype(np.float64), pos, cache, mode="own")
        check_rows(out.cpu().numpy(), x, ref, 1e-4, ("f32", shift, i))
        if i == 2:  # (one row takes the decode attention, another split)
            dm.sublayer_apply(i, xd[17:18].contiguous(), pos[17:18], mode=1, out=one)
            assert torch.equal(one[0], out[17])
    logits, _, _ = dm.head_rows(torch.from_numpy(x).cuda())
    assert rel_err(logits.cpu().numpy(), M.head(model, x.astype(np.float64))[0]) < 1e-4
    dm.close()


# one instance of the walking kernel per d / 1024; the 8B decoders' is the last
@pytest.mark.parametrize("d", [1024, 2048, 3072, 4096])
def test_head_rows_keep_their_bits(d):
    """A large vocabulary (65552: 4097 tiles, one more than 16 rounds of 256
    workgroups): 4 to 8 rows run on workgroups that walk the tiles, 1 to 3 and 9 to
    16 on one tile each; a row's logits are the same bits in all of them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd.engine import DeviceModel
    cfg = dataclasses.replace(W.config("small_bf16"), name="head_bf16", L=1, d=d, hq=2, hkv=1,
                              ffn=32, vocab=65552)
    w = W.generate_weights(cfg, seed=0)
    dm = DeviceModel(cfg, n_max=64, gamma_max=15, cap_max=16, prefill_chunk=16).upload_all(w)
    x = torch.from_numpy(W.synthetic_rows(12, d, seed=4, std=0.5, index=11)).cuda()
    all_rows = dm.head_rows(x)[0]
    for a, b in ((0, 1), (1, 4), (4, 8), (3, 8), (4, 12), (0, 7)):
        logits, am, _ = dm.head_rows(x[a:b].contiguous())
        assert torch.equal(logits, all_rows[a:b]), (a, b)
        assert torch.equal(am.long(), logits.argmax(-1))
    lg0 = M.head(M.Model(cfg, w), x[4:6].cpu().numpy().astype(np.float64))[0]
    assert rel_err(all_rows[4:6].cpu().numpy(), lg0) < TOL
    dm.close()


def test_head_rows_of_one_row_tile():
    """65552 columns: up to 128 rows take 128 x 128 tiles, the last of them with one
    column tile of eight, 129 rows a wider tile; a row's logits are the same bits
    in all of them (32 rows and more: no K split at 1024)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_20217_amd.engine import DeviceModel
    cfg = dataclasses.replace(W.config("small_bf16"), name="head_bf16", L=1, d=1024, hq=2, hkv=1,
                              ffn=32, vocab=65552)
    w = W.generate_weights(cfg, seed=0)
    dm = DeviceModel(cfg, n_max=64, gamma_max=15, cap_max=16, prefill_chunk=16).upload_all(w)
    x = torch.from_numpy(W.synthetic_rows(300, 1024, seed=4, std=0.5, index=12)).cuda()
    all_rows = dm.head_rows(x)[0]
    for a, b in ((0, 32), (5, 69), (100, 228), (100, 229)):
        logits, am, _ = dm.head_rows(x[a:b].contiguous())
        assert torch.equal(logits, all_rows[a:b]), (a, b)
        assert torch.equal(am.long(), logits.argmax(-1))
    s = [0, 16, 127, 128, 299]
    lg0 = M.head(M.Model(cfg, w), x[s].cpu().numpy().astype(np.float64))[0]
    assert rel_err(all_rows[s].cpu().numpy(), lg0) < TOL
    dm.close()

"""Passes of more than 80 rows (the tiled GEMM, gemm_tile.hip) against the same
rows in passes of at most 80 (the skinny kernels, which the oracle tests cover
at full widths): one layer of the 36-layer shapes under a head of 33 128-id
blocks.  Row counts sit at the edges of the row tiles (128, 192, 256) and of the
first row count that takes them.  (These sizes take five of the six tiles;
test_gpu_gemm.py runs every kernel by itself, half-empty tiles among them.)
Both sides sum in fp32 over the same bf16 rounding points: they differ where a
value falls on the other side of a rounding, within the bound the oracle
comparison uses for up to two layers (5e-2 on the logits, 3e-2 on K and V)."""
import numpy as np
import pytest
import torch

from paper_2607_17299_amd import harness, synth
from parity import LOGIT_TOL

pytestmark = pytest.mark.gpu
CFG = synth.reduced(synth.LARGE, 1, vocab=33 * 128)
DEV = "cuda"


@pytest.fixture(scope="module")
def models():
    from paper_2607_17299_amd import war
    w = harness.large_weights(CFG)
    return {"war": war, "many": war.Model(CFG, w, max_rows=1024), "few": war.Model(CFG, w, max_rows=80)}


def _t(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.int32).to(DEV)


@pytest.mark.parametrize("rows", [81, 96, 128, 129, 192, 193, 257, 513, 1000])
def test_append_rows_match_small_passes(models, rows):
    war = models["war"]
    lens = [rows - rows // 3, rows // 3]                 # two sequences share the passes
    toks = np.concatenate([synth.uniform_tokens(40 + i, n, CFG.vocab) for i, n in enumerate(lens)])
    out = {}
    for name in ("many", "few"):
        pool = war.Pool(CFG, 2 * (rows // 16 + 2), 2, rows // 16 + 2)
        pool.kv.zero_()
        logits = torch.zeros((2, CFG.vocab), device=DEV)
        war.prefill_append(models[name], pool, _t([0, 1]), _t([0, 0]), lens, _t(toks), _t([0, 0]), logits)
        torch.cuda.synchronize()
        out[name] = (logits, [pool.gather_kv(s, n, 0).float() for s, n in enumerate(lens)])
    assert (out["many"][0] - out["few"][0]).abs().max() <= LOGIT_TOL
    for a, b in zip(out["many"][1], out["few"][1]):
        assert torch.allclose(a, b, atol=3e-2, rtol=2e-2)


@pytest.mark.parametrize("B,k", [(27, 2), (43, 2), (64, 2), (65, 2), (128, 1), (171, 2)])
def test_verify_rows_match_small_steps(models, B, k):
    """B * (k + 1) = 81 .. 513 rows, against steps of at most 20 requests."""
    war = models["war"]
    pool = war.Pool(CFG, B * 4, B, 4)
    ctx = [3 + (5 * b) % 37 for b in range(B)]
    harness.load_contexts(pool, CFG, ctx, list(range(B)), kv_seed=3)
    rng = np.random.default_rng(B)
    last, drafts = rng.integers(0, CFG.vocab, B), rng.integers(0, CFG.vocab, (B, k))

    def step(model, lo, hi):
        n = hi - lo
        acc, nxt = _t([0] * n), _t([0] * n)
        logits = torch.zeros((n * (k + 1), CFG.vocab), device=DEV)
        war.verify_step(model, pool, _t(range(lo, hi)), _t(ctx[lo:hi]), _t(last[lo:hi]), _t(drafts[lo:hi]), None, k,
                        acc, nxt, logits)
        war.kv_commit(pool, _t(range(lo, hi)), _t(ctx[lo:hi]), _t([-1] * n))
        torch.cuda.synchronize()
        return logits, acc, nxt

    big = step(models["many"], 0, B)
    small = [step(models["few"], lo, min(B, lo + 20)) for lo in range(0, B, 20)]
    ref = torch.cat([s[0] for s in small])
    err = (big[0] - ref).abs().amax(1)
    assert err.max() <= LOGIT_TOL
    # the fused argmax is the argmax of the logits it wrote, lowest id first
    rows = big[0].view(B, k + 1, -1)
    greedy = (rows == rows.amax(-1, keepdim=True)).int().argmax(-1).cpu().numpy()
    for b in range(B):
        a = 0
        while a < k and drafts[b][a] == greedy[b, a]:
            a += 1
        assert (int(big[1][b]), int(big[2][b])) == (a, greedy[b, a])


# one layer of narrow matrices: splits of one and two k-steps, a residual of more
# than eight splits over rows of 1024 (four thread groups), 768 (five) and 2048 (two)
@pytest.mark.parametrize("d,heads,ffn", [(1024, 16, 4096), (768, 12, 3072), (2048, 16, 2048)])
@pytest.mark.parametrize("B,k", [(1, 0), (4, 3), (11, 2), (8, 5), (11, 5), (16, 4)])
def test_narrow_matrices_match_oracle(d, heads, ffn, B, k):
    from oracle.decoder import RequestKV, Weights
    from oracle.verify import verify_request
    from paper_2607_17299_amd import war
    cfg = synth.ModelConfig(n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=heads // 4, head_dim=64, ffn_dim=ffn,
                            vocab=1024)
    w = synth.model_weights(cfg, seed=1, norm_std=0.1)
    model, W = war.Model(cfg, {n: t.to(DEV) for n, t in w.items()}, max_rows=80), Weights(cfg, w)
    ctx = [1 + (7 * b) % 23 for b in range(B)]
    pool = war.Pool(cfg, B * 4, B, 4)
    harness.load_contexts(pool, cfg, ctx, list(range(B)), kv_seed=4)
    rng = np.random.default_rng(B + k)
    last, drafts = rng.integers(0, cfg.vocab, B), rng.integers(0, cfg.vocab, (B, max(k, 1)))
    acc, nxt = _t([0] * B), _t([0] * B)
    logits = torch.zeros((B * (k + 1), cfg.vocab), device=DEV)
    war.verify_step(model, pool, _t(range(B)), _t(ctx), _t(last), _t(drafts), None, k, acc, nxt, logits)
    torch.cuda.synchronize()
    got = logits.cpu().numpy().reshape(B, k + 1, -1)
    for b in range(0, B, 3):
        kv = synth.kv_context(cfg, 4, b, 0, 0, ctx[b], DEV).cpu().double().numpy()
        r = verify_request(cfg, W, RequestKV(cfg, [(kv[0], kv[1])]), int(last[b]), drafts[b][:k].tolist())
        assert np.abs(r["logits"] - got[b]).max() <= LOGIT_TOL


@pytest.mark.parametrize("rows", [81, 96, 97])
@pytest.mark.parametrize("d", [256, 1024, 4096])      # loops of 4 k-steps, and 16 and 64 unrolled
def test_large_lm_head_rows_match_small_steps(rows, d):
    """A head of 257 128-id blocks at the row counts where its kernel changes,
    against the same requests in steps of 27: the rows' logits and argmax."""
    from paper_2607_17299_amd import war
    cfg = synth.ModelConfig(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=2, head_dim=128, ffn_dim=256,
                            vocab=257 * 128)
    g = torch.Generator(device=DEV).manual_seed(d)
    w = {n: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0, 0.02 if len(s) > 1 else 0.5, generator=g)
         for n, s in synth.weight_shapes(cfg)}
    model, pool = war.Model(cfg, w, max_rows=128), war.Pool(cfg, rows, rows, 2)
    last = np.random.default_rng(d).integers(0, cfg.vocab, rows)

    def step(lo, hi):
        n = hi - lo
        acc, nxt, logits = _t([0] * n), _t([0] * n), torch.zeros((n, cfg.vocab), device=DEV)
        war.verify_step(model, pool, _t(range(lo, hi)), _t([0] * n), _t(last[lo:hi]), None, None, 0, acc, nxt, logits)
        war.kv_commit(pool, _t(range(lo, hi)), _t([0] * n), _t([-1] * n))
        torch.cuda.synchronize()
        return logits, nxt

    got = step(0, rows)
    ref = torch.cat([step(lo, min(rows, lo + 27))[0] for lo in range(0, rows, 27)])
    assert (got[0] - ref).abs().max() <= LOGIT_TOL
    assert torch.equal(got[1].long(), (got[0] == got[0].amax(-1, keepdim=True)).int().argmax(-1))


def test_append_metadata_grows_in_few_steps():
    """A trajectory that gets a little longer with every append: the metadata block
    is allocated a few times in all, not at every turn."""
    import ctypes as C

    from paper_2607_17299_amd import war
    cfg = synth.reduced(synth.TINY, 1)
    w = {n: t.to(DEV) for n, t in synth.model_weights(cfg, seed=0, norm_std=0.1).items()}
    model, pool = war.Model(cfg, w, max_rows=4096), war.Pool(cfg, 4000, 1, 4000)
    ctx, nxt, sizes = _t([0]), _t([0]), set()
    for turn in range(1, 64):
        n = 7 * turn
        war.prefill_append(model, pool, _t([0]), ctx, [n], _t(np.arange(n) % cfg.vocab), nxt)
        p, size = C.c_void_p(), C.c_int64()
        assert war.lib().war_debug_workspace(model.handle, b"stage", C.byref(p), C.byref(size)) == 0
        sizes.add(size.value)
    assert int(ctx[0]) == 7 * 63 * 32 and len(sizes) <= 2
    n = 4 * 4096 - 100                     # more rows than any append before it
    war.prefill_append(model, pool, _t([0]), ctx, [n], _t(np.arange(n) % cfg.vocab), nxt)
    torch.cuda.synchronize()
    assert war.lib().war_debug_workspace(model.handle, b"stage", C.byref(p), C.byref(size)) == 0
    assert size.value >= 2 * max(sizes) or size.value == max(sizes)

"""The prefill attention (attn_rows.hip) at the edges of what it walks: key blocks
of 32, chunks of 4096 keys, vectors of 64 page ids (1024 keys), row blocks of 128
rows.  Appends over cached contexts, on a pool whose every slot starts as NaN, so
that a slot past a sequence's end which reached a product would show, against the
same tokens taken by verify steps of at most 48 rows (those the oracle tests
cover).  Both layers' new keys and values are compared, the second layer's of
every new row depending on that row's attention in the first, and the logits after
the last token.  Queries and keys are large enough that each row rests on a few
keys, wherever these lie.  The two sum in different orders: they differ where a value falls
on the other side of a bf16 rounding, within the bounds the oracle comparison uses
for two layers (5e-2 on the logits, 3e-2 on K and V)."""
import numpy as np
import pytest
import torch

from paper_2607_17299_amd import synth
from parity import LOGIT_TOL

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _t(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.int32).to(DEV)


@pytest.fixture(scope="module")
def models():
    from paper_2607_17299_amd import war
    out = {}
    for G, hd in [(4, 128), (4, 64), (1, 64), (8, 128), (2, 64)]:
        cfg = synth.ModelConfig(n_layers=2, d_model=256, n_q_heads=2 * G * 64 // hd if G * hd < 1024 else 8,
                                n_kv_heads=2 * 64 // hd if G * hd < 1024 else 1, head_dim=hd, ffn_dim=512, vocab=1024)
        assert cfg.group == G
        w = {n: t.to(DEV) for n, t in synth.model_weights(cfg, seed=3, norm_std=0.1).items()}
        for l in range(2):
            w[f"l{l}.w_qkv"] *= 6                  # queries, keys and values of std 2
        out[G, hd] = (cfg, war.Model(cfg, w, max_rows=512))
    return war, out


def _pool(war, cfg, ctx, n_new):
    total = [c + n for c, n in zip(ctx, n_new)]
    pool = war.Pool(cfg, sum(n // 16 + 2 for n in total), len(ctx), max(total) // 16 + 5)
    pool.kv.fill_(float("nan"))
    pool.alloc(list(range(len(ctx))), ctx)
    for s, c in enumerate(ctx):
        for l in range(cfg.n_layers if c else 0):
            pool.load(s, l, 0, 2 * synth.kv_context(cfg, 6, s, l, 0, c, DEV))
    torch.cuda.synchronize()
    return pool


def _append(war, cfg, model, ctx, toks):
    pool = _pool(war, cfg, ctx, [len(t) for t in toks])
    logits, lens = torch.zeros((len(ctx), cfg.vocab), device=DEV), _t(ctx)
    war.prefill_append(model, pool, _t(range(len(ctx))), lens, [len(t) for t in toks], _t(np.concatenate(toks)),
                       _t([0] * len(ctx)), logits)
    return pool, logits


def _by_steps(war, cfg, model, ctx, toks):
    """The same tokens as verify steps whose drafts are all kept."""
    pool, kp1 = _pool(war, cfg, ctx, [len(t) for t in toks]), min(48 // cfg.group, 12)
    last, done = torch.zeros((len(ctx), cfg.vocab), device=DEV), 0
    while True:
        live = [s for s in range(len(ctx)) if len(toks[s]) > done]
        if not live:
            return pool, last
        part = [toks[s][done:done + kp1] for s in live]
        B, k = len(live), kp1 - 1
        drafts = np.zeros((B, max(k, 1)), np.int64)
        for b, p in enumerate(part):
            drafts[b, :len(p) - 1] = p[1:]
        lens = _t([ctx[s] + done for s in live])
        logits, acc, nxt = torch.zeros((B * kp1, cfg.vocab), device=DEV), _t([0] * B), _t([0] * B)
        war.verify_step(model, pool, _t(live), lens, _t([p[0] for p in part]), _t(drafts),
                        _t([len(p) - 1 for p in part]), k, acc, nxt, logits)
        war.kv_commit(pool, _t(live), lens, _t([len(p) - 1 for p in part]))
        torch.cuda.synchronize()
        for b, s in enumerate(live):
            last[s] = logits[b * kp1 + len(part[b]) - 1]
        done += kp1


def _compare(models, shape, ctx, n_new):
    war, by_shape = models
    cfg, model = by_shape[shape]
    toks = [synth.uniform_tokens(70 + s, n, cfg.vocab) for s, n in enumerate(n_new)]
    got, ref = _append(war, cfg, model, ctx, toks), _by_steps(war, cfg, model, ctx, toks)
    torch.cuda.synchronize()
    assert torch.isfinite(got[1]).all() and torch.isfinite(ref[1]).all()
    assert (got[1] - ref[1]).abs().max() <= LOGIT_TOL
    for s, (c, n) in enumerate(zip(ctx, n_new)):
        for l in range(cfg.n_layers):
            a, b = (p.gather_kv(s, c + n, l)[:, :, c:].float() for p in (got[0], ref[0]))
            assert torch.isfinite(a).all()
            assert torch.allclose(a, b, atol=3e-2, rtol=2e-2), (s, l)


SHAPES = [(4, 128), (4, 64), (1, 64), (8, 128), (2, 64)]


@pytest.mark.parametrize("shape", SHAPES)
def test_first_blocks(models, shape):
    """No cached keys: 1 to 5 blocks, every kind of last block (S % 32 of 0, 1, 15,
    16, 17 and 31), one sequence each, all in one append."""
    n_new = [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 128, 129, 144, 160]
    _compare(models, shape, [0] * len(n_new), n_new)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("base", [1024, 2048, 4096, 8192])
def test_page_vector_and_chunk_edges(models, shape, base):
    """Sequences that end around a multiple of 1024 keys (a new vector of page ids)
    and of 4096 (a new chunk of 1 to 5 blocks), few and many new rows."""
    ends = [base - 1, base, base + 1, base + 31, base + 33, base + 64, base + 111, base + 160]
    n_new = [3, 40, 1, 17, 33, 65, 130, 161]
    _compare(models, shape, [e - n for e, n in zip(ends, n_new)], n_new)


@pytest.mark.parametrize("shape", SHAPES)
def test_rows_over_many_blocks(models, shape):
    """More new rows than a pass holds (512), so that blocks above the causal line and
    rows beyond a row block's end occur with every alignment."""
    _compare(models, shape, [0, 13, 1000], [700, 345, 27])

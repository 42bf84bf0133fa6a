"""How a verify step cuts its keys into attention units: a step too small for
the grid takes chunks of 512, 256 or 128 keys, which must give what 1024-key
chunks give (those the oracle tests cover).  A pool with forked sequences keeps
1024-key chunks, so the same step runs there as the reference.  Both merge fp32
partials of the same bf16 products; they differ where a value falls on the other
side of a rounding, within the bound the oracle comparison uses."""
import numpy as np
import pytest
import torch

from paper_2607_17299_amd import harness, synth
from parity import LOGIT_TOL

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _t(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.int32).to(DEV)


@pytest.fixture(scope="module")
def models():
    from paper_2607_17299_amd import war
    out = {}
    for name, cfg in (("large", synth.reduced(synth.LARGE, 1, vocab=1024)), ("tiny", synth.TINY)):
        if name == "large":
            w = harness.large_weights(cfg)
        else:
            w = {k: v.to(DEV) for k, v in synth.model_weights(cfg, seed=0, norm_std=0.1).items()}
        out[name] = (cfg, war.Model(cfg, w, max_rows=256))
    return war, out


# (shape, contexts, drafts, keys per item); 8 kv-heads fill at 64 items, 2 at 256
@pytest.mark.parametrize("shape,ctx,k,chunk", [
    ("large", [1023], 0, 1024), ("large", [1024], 0, 128), ("large", [1500], 11, 128), ("large", [8191], 0, 128),
    ("large", [8192], 0, 256), ("large", [16384], 4, 512), ("large", [3000, 17, 1], 8, 128),
    ("large", [4000] * 7, 3, 512), ("large", [9000] * 7, 2, 1024),
    ("tiny", [512, 505, 498], 4, 1024), ("tiny", [1030, 3], 23, 128), ("tiny", [5000] * 9, 5, 256)])
def test_short_chunks_match_whole_ones(models, shape, ctx, k, chunk):
    war, by_name = models
    cfg, model = by_name[shape]
    B = len(ctx)
    rng = np.random.default_rng(B + k)
    last, drafts = rng.integers(0, cfg.vocab, B), rng.integers(0, cfg.vocab, (B, max(k, 1)))
    got = {}
    for forked in (False, True):
        pool = war.Pool(cfg, sum(c // 16 + 4 for c in ctx) + 4, B + 3, max(ctx) // 16 + 8)
        harness.load_contexts(pool, cfg, ctx, list(range(B)), kv_seed=9)
        seqs, lens, pend, dr = list(range(B)), list(ctx), list(last), list(drafts)
        if forked:                  # two spare sequences sharing a page, and a batch of two or more
            pool.alloc([B], [16])
            pool.fork(B, B + 1, 16)
            if B == 1:
                seqs, lens, pend, dr = [0, B + 2], [ctx[0], 0], [last[0], 0], [drafts[0], drafts[0]]
        n = len(seqs)
        acc, nxt = _t([0] * n), _t([0] * n)
        logits = torch.zeros((n * (k + 1), cfg.vocab), device=DEV)
        war.verify_step(model, pool, _t(seqs), _t(lens), _t(pend), _t(np.stack(dr)), None, k, acc, nxt, logits)
        torch.cuda.synchronize()
        keys = war.debug_workspace(model, "n_items", torch.int32, (4,)).cpu().tolist()[3]
        assert keys == (1024 if forked else chunk)
        got[forked] = logits[:B * (k + 1)]
    assert torch.isfinite(got[False]).all()
    assert (got[False] - got[True]).abs().max() <= LOGIT_TOL


def _plan(war, model, pool, lens, k):
    """Items, work order, units and keys per item of a step over sequences 0 .. B-1."""
    B = len(lens)
    acc, nxt = _t([0] * B), _t([0] * B)
    war.verify_step(model, pool, _t(range(B)), _t(lens), _t([1] * B), _t(np.ones((B, max(k, 1)))), None, k, acc, nxt)
    war.kv_commit(pool, _t(range(B)), _t(lens), _t([-1] * B))
    torch.cuda.synchronize()
    get = lambda name, shape: war.debug_workspace(model, name, torch.int32, shape).cpu().numpy()
    n_items, n_units, _, chunk = get("n_items", (4,)).tolist()
    return get("items", (n_items, 4)), get("order", (n_units,)), n_units, chunk


@pytest.mark.parametrize("B", [1, 2, 17, 64, 65, 128])
def test_work_order_of_an_unforked_batch(models, B):
    """Whole chunks in request order, then the partial ones, longest first."""
    war, by_name = models
    cfg, model = by_name["tiny"]
    rng = np.random.default_rng(B)
    lens = [int(x) for x in rng.choice([0, 1, 127, 1023, 1024, 2047, 2048, 3000, 4095], B)]
    pool = war.Pool(cfg, sum(c // 16 + 2 for c in lens), B, 260)
    pool.kv.zero_()
    pool.alloc(list(range(B)), lens)
    items, order, n_units, chunk = _plan(war, model, pool, lens, 0)
    keys = [n + 1 for n in lens]
    want = [[b, 0, c, 0] for b, n in enumerate(keys) for c in range(-(-n // chunk))]
    assert items.tolist() == want and n_units == len(want)
    whole = [i for i, (b, _, c, _) in enumerate(want) if (c + 1) * chunk <= keys[b]]
    part = [i for i, (b, _, c, _) in enumerate(want) if (c + 1) * chunk > keys[b]]
    part.sort(key=lambda i: (-(keys[want[i][0]] % chunk), want[i][0]))
    assert order.tolist() == whole + part


@pytest.mark.parametrize("pages", [1, 63, 64, 65, 127, 511, 512, 513, 576])
def test_shared_pages_of_forked_siblings(models, pages):
    """Three siblings with `pages` pages in common and a stranger: the 1024-key
    chunks inside them are attended once for all three."""
    war, by_name = models
    cfg, model = by_name["tiny"]
    lens = [pages * 16 + 40, pages * 16 + 3, pages * 16 + 200, 700]
    pool = war.Pool(cfg, 3 * pages + 120, 4, pages + 60)
    pool.kv.zero_()
    pool.alloc([0], [lens[0]])
    for s in (1, 2):
        pool.fork(0, s, pages * 16)
    pool.alloc([1, 2, 3], lens[1:])
    items, order, n_units, chunk = _plan(war, model, pool, lens, 0)
    shared = pages * 16 // 1024
    n = [-(-(x + 1) // 1024) for x in lens]
    assert chunk == 1024 and n_units == sum(n) - 2 * shared
    own = {0: 3, 1: -1, 2: -1, 3: 0}
    assert items.tolist() == [[b, 0, c, own[b] if c < shared else 0] for b in range(4) for c in range(n[b])]
    assert sorted(order.tolist()) == [i for i, it in enumerate(items.tolist()) if it[3] >= 0]


@pytest.mark.parametrize("heads,kv", [(6, 3), (12, 6), (10, 5), (24, 24)])
def test_shortened_chunks_fit_the_grid(heads, kv):
    """Chunks are shortened while the units (items times kv-heads) are no more than
    the grid's 512 workgroups, also where the kv-heads do not divide 512."""
    from paper_2607_17299_amd import war
    cfg = synth.ModelConfig(n_layers=1, d_model=128 * heads // 2, n_q_heads=heads, n_kv_heads=kv, head_dim=64,
                            ffn_dim=256, vocab=1024)
    w = {n: t.to(DEV) for n, t in synth.model_weights(cfg, seed=2, norm_std=0.1).items()}
    model = war.Model(cfg, w, max_rows=64)
    fill = 512 // kv
    shortened = 0
    for B in (1, 3):
        pool = war.Pool(cfg, B * 1700, B, 1700)
        pool.kv.zero_()
        pool.alloc(list(range(B)), [26000] * B)
        for items in (fill - 1, fill, fill + 1, 2 * fill + 1):
            for chunk in (128, 256, 512):
                n = min(items // B * chunk, 26000) - 1
                lens = [n] + [n - 7] * (B - 1)
                if n < 1024:
                    continue
                got, _, n_units, keys = _plan(war, model, pool, lens, 0)
                assert n_units == len(got) and keys in (128, 256, 512, 1024)
                if keys < 1024:
                    shortened += 1
                    assert n_units * kv <= 512, (lens, keys)
        pool.close()
    assert shortened >= 4


@pytest.mark.parametrize("lens,keys", [
    ([8191], 128), ([8192], 256), ([16000], 256), ([16384], 512), ([32767], 512), ([32768], 1024), ([60000], 1024),
    ([16000, 3], 256), ([20000, 19000, 5], 512), ([3, 40000], 1024), ([2000] * 4, 128)])
def test_shortened_chunks_leave_at_most_64_partials(lens, keys):
    """One kv-head: 512 items fill the grid, but a request is cut into at most 64."""
    from paper_2607_17299_amd import war
    cfg = synth.ModelConfig(n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=256, vocab=1024)
    w = {n: t.to(DEV) for n, t in synth.model_weights(cfg, seed=2, norm_std=0.1).items()}
    model, B = war.Model(cfg, w, max_rows=64), len(lens)
    pool = war.Pool(cfg, sum(n // 16 + 2 for n in lens), B, max(lens) // 16 + 2)
    pool.kv.zero_()
    pool.alloc(list(range(B)), lens)
    items, _, _, got = _plan(war, model, pool, lens, 0)
    assert got == keys and len(items) == sum(-(-(n + 1) // keys) for n in lens)


@pytest.mark.parametrize("shape,k", [("tiny", 1), ("tiny", 2), ("tiny", 4), ("tiny", 8), ("large", 1), ("large", 2),
                                     ("large", 4), ("large", 8)])
def test_shared_pages_of_siblings_with_drafts(models, shape, k):
    """Five siblings with full drafts: a run holds as many consecutive members as have
    their rows fit the step's row block together (with more drafts, one), its first
    member owns the shared chunks, each run's once."""
    from parity import shared_units
    war, by_name = models
    cfg, model = by_name[shape]
    pages, B, G = 130, 5, cfg.group
    lens = [pages * 16 + n for n in (40, 3, 200, 77, 12)]
    pool = war.Pool(cfg, B * (pages + 20), B, pages + 60)
    pool.kv.zero_()
    pool.alloc([0], [lens[0]])
    for s in range(1, B):
        pool.fork(0, s, pages * 16)
    pool.alloc(list(range(1, B)), lens[1:])
    items, order, n_units, chunk = _plan(war, model, pool, lens, k)
    rows = G * (k + 1)
    runs = shared_units([rows] * B, 16 if rows <= 16 else 32 if rows <= 32 else 48)
    own = [x for r in runs for x in [r] + [-1] * (r - 1)]
    shared, n = pages * 16 // 1024, [-(-(x + k + 1) // 1024) for x in lens]
    assert chunk == 1024 and n_units == sum(n) - (B - len(runs)) * shared
    assert items.tolist() == [[b, 0, c, own[b] if c < shared else 0] for b in range(B) for c in range(n[b])]
    assert sorted(order.tolist()) == [i for i, it in enumerate(items.tolist()) if it[3] >= 0]

"""GPU parity of the sampled-verification decision kernels on seeded synthetic
logit rows (war_debug_sample runs them alone), against the oracle's rule on
the very same rows and uniforms.  The kernels decide in fp32 and the oracle in
float64, so a decision may differ only where its margin is below 1e-5
(reported)."""
import numpy as np
import pytest
import torch

from oracle.sampling import filtered_probs, verify_sampled

pytestmark = pytest.mark.gpu


def _case(V, B, k, T, top_k, scale, seed, ties=False, alter=None):
    from paper_2607_17299_amd import war
    rng = np.random.default_rng(seed)
    z = (rng.standard_normal((B * (k + 1), V)) * scale).astype(np.float32)
    if alter:
        alter(z, rng)
    if ties:
        # exact ties at the top_k boundary and at the maximum
        for r in range(z.shape[0]):
            order = np.argsort(-z[r].astype(np.float64), kind="stable")
            kth = z[r, order[top_k - 1]]
            z[r, rng.choice(V, 5, replace=False)] = kth
            z[r, rng.choice(V, 2, replace=False)] = z[r].max()
    dls = rng.integers(0, k + 1, B)
    drafts = np.zeros((B, max(k, 1)), np.int32)
    for b in range(B):
        for i in range(dls[b]):
            p = filtered_probs(z[b * (k + 1) + i].astype(np.float64), T, top_k)
            # likely tokens (drawn from the target) and, sometimes, unlikely ones
            drafts[b, i] = rng.choice(V, p=p) if rng.random() < 0.8 else rng.integers(V)
    u = rng.random((B * (k + 1), 2)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    acc = torch.zeros(B, dtype=torch.int32, device="cuda")
    nxt = torch.zeros(B, dtype=torch.int32, device="cuda")
    war.debug_sample(dev(z), dev((dls + 1).astype(np.int32)), dev(drafts), k, dev(u), T, top_k, acc, nxt)
    acc, nxt = acc.cpu().numpy(), nxt.cpu().numpy()
    exact, report, n_acc = 0, [], 0
    for b in range(B):
        n = int(dls[b])
        rows = z[b * (k + 1): b * (k + 1) + n + 1].astype(np.float64)
        uu = u[b * (k + 1): b * (k + 1) + n + 1].astype(np.float64)
        r = verify_sampled(rows, drafts[b, :n].tolist(), uu[:, 0], uu[:, 1], T, top_k)
        n_acc += r["accept"]
        if (int(acc[b]), int(nxt[b])) == (r["accept"], r["next"]):
            exact += 1
        else:
            assert min(r["margins"]) < 1e-5, (b, (int(acc[b]), int(nxt[b])), (r["accept"], r["next"]), r["margins"])
            report.append(b)
    return exact, report, n_acc


@pytest.mark.parametrize("V,T,top_k,scale", [
    (151936, 1.0, 200, 1.0),     # the paper's setting on the 36-layer vocabulary
    (151936, 1.0, 200, 6.0),     # peaked rows: drafts are often accepted
    (4096, 0.7, 50, 3.0),
    (4096, 1.5, 4096, 2.0),      # top_k = vocabulary: plain temperature sampling
    (4096, 1.0, 1, 1.0),         # greedy
])
def test_sampling_kernels_match_the_rule(V, T, top_k, scale):
    exact, report, n_acc = _case(V, 24, 4, T, top_k, scale, seed=V + top_k + int(10 * scale))
    assert exact + len(report) == 24 and len(report) <= 1, report
    print(f"\nV={V} T={T} top_k={top_k}: {exact}/24 exact, accepted drafts {n_acc}, reported {report}")


def test_sampling_kernels_ties_at_the_boundary():
    """Exact ties at the top_k boundary (kept by lowest id) and at the maximum."""
    exact, report, _ = _case(4096, 24, 4, 1.0, 200, 2.0, seed=99, ties=True)
    assert exact + len(report) == 24 and len(report) <= 1, report


def _signed_zeros(z, rng):
    """Everything kept is +0 or -0 (one value): ties by id across block maxima."""
    z[:] = np.where(rng.random(z.shape) < 0.01, np.where(rng.random(z.shape) < 0.5, 0.0, -0.0), -1.0 - np.abs(z))


def _one_block(z, rng):
    """Every large logit in one 128-id block: the other blocks' maxima set the bound."""
    z[:, 256:384] += 30.0


def _equal(z, rng):
    z[:] = 1.5        # more candidates than a workgroup holds: the row path


def _infinite(z, rng):
    z[rng.random(z.shape) < 0.9] = -np.inf


@pytest.mark.parametrize("V,top_k,alter", [
    (151936, 1187, None),          # as many kept ids as 128-id blocks
    (151936, 1188, None),          # one more: the row path
    (128, 1, None), (384, 3, None),
    (4096 * 128, 200, None),       # the most blocks a workgroup handles
    (4097 * 128, 200, None),       # one more: the row path
    (4096 + 64, 20, None),         # not whole blocks: the row path
    (32768, 200, _signed_zeros), (32768, 100, _one_block), (32768, 200, _equal), (32768, 256, _infinite),
])
def test_sampling_block_bound_edges(V, top_k, alter):
    """The block-maximum path and its limits give the rule's decisions (margins
    below 1e-5, fp32 sums against float64, are reported)."""
    exact, report, _ = _case(V, 4, 2, 1.0, top_k, 2.0, seed=V + top_k, alter=alter)
    assert exact + len(report) == 4 and len(report) <= 1, report


def _nan_rule(z, d, u, v, top_k):
    """(accepted?, token if rejected here, token if last) of a row that may hold
    NaNs: a positive one sorts above every number and is kept, a negative one
    below.  A kept NaN makes the total weight NaN: no draft is accepted and no
    cumulative weight exceeds the target, which leaves the highest kept id (other
    than a rejected draft) of nonzero weight."""
    bits = (z + np.float32(0)).view(np.uint32)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(0x80000000))
    kept = np.sort(np.lexsort((np.arange(z.size), -key.astype(np.int64)))[:top_k])
    if np.isnan(z[kept]).any():
        live = kept[~np.isnan(z[kept])]
        return False, int(live[live != d].max()), int(live.max())
    clean = np.where(np.isnan(z), -np.inf, z).astype(np.float64)
    r = verify_sampled(np.stack([clean, clean]), [int(d)] if d >= 0 else [], [u, u], [v, v], 1.0, top_k)
    end = verify_sampled(clean[None], [], [u], [v], 1.0, top_k)["next"]
    return bool(r["accept"]) and d >= 0, r["next"], end


def _decide(rows, drafts, u, top_k):
    for i in range(len(rows)):
        d = drafts[i] if i < len(drafts) else -1
        ok, rej, end = _nan_rule(rows[i], d, u[i, 0], u[i, 1], top_k)
        if i < len(drafts) and ok:
            continue
        return i, rej if i < len(drafts) else end


@pytest.mark.parametrize("where", ["best block", "worst block", "several"])
@pytest.mark.parametrize("sign", [1, -1])
def test_sampling_rows_with_nan(where, sign):
    """A NaN logit, in a block that the block maxima select, in one that they do
    not, in each lane of both halves of a block: the decisions of the row walk."""
    from paper_2607_17299_amd import war
    V, B, k, top_k = 8192, 64, 1, 20
    rng = np.random.default_rng(11)
    z = (rng.standard_normal((B * (k + 1), V)) * 2).astype(np.float32)
    nan = np.array([0x7fc00000 if sign > 0 else 0xffc00000], np.uint32).view(np.float32)[0]
    for r in range(z.shape[0]):
        best = z[r].reshape(-1, 128).max(1).argsort()
        blk = best[-1] if where == "best block" else best[0]
        z[r, blk * 128 + r] = nan                       # B * (k + 1) = 128 rows: every position once
        if where == "several":
            z[r, rng.choice(V, 3, replace=False)] = nan
    drafts = z[::2].argsort(1)[:, -2:-1].astype(np.int32)
    u = rng.random((B * (k + 1), 2)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    acc, nxt = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
    war.debug_sample(dev(z), dev(np.full(B, k + 1, np.int32)), dev(drafts), k, dev(u), 1.0, top_k, acc, nxt)
    got = list(zip(acc.cpu().tolist(), nxt.cpu().tolist()))
    want = [_decide(z[2 * b: 2 * b + 2], drafts[b].tolist(), u[2 * b: 2 * b + 2], top_k) for b in range(B)]
    assert got == want


@pytest.mark.parametrize("B", [4, 40])               # 12 and 120 rows: both LM-head kernels
@pytest.mark.parametrize("col", [0, 17, 63, 100, 127])
def test_sampled_step_with_a_nan_column(B, col):
    """A NaN weight in one LM-head row: every row's logits hold one NaN."""
    from paper_2607_17299_amd import harness, synth, war
    cfg, k, top_k = synth.reduced(synth.TINY, 1), 2, 20
    w = {n: t.cuda() for n, t in synth.model_weights(cfg, seed=0, norm_std=0.1).items()}
    w["w_lm"][5 * 128 + col, 3] = float("nan")
    model, pool = war.Model(cfg, w, max_rows=128), war.Pool(cfg, 2 * B, B, 2)
    t = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.int32).cuda()
    ctx = [1 + b % 20 for b in range(B)]
    harness.load_contexts(pool, cfg, ctx, list(range(B)), kv_seed=3)
    rng = np.random.default_rng(B)
    drafts, u = rng.integers(0, cfg.vocab, (B, k)), rng.random((B * (k + 1), 2)).astype(np.float32)
    acc, nxt, logits = t([0] * B), t([0] * B), torch.zeros((B * (k + 1), cfg.vocab), device="cuda")
    war.verify_step_sampled(model, pool, t(range(B)), t(ctx), t(rng.integers(0, cfg.vocab, B)), t(drafts), None, k,
                            torch.from_numpy(u).cuda(), 1.0, top_k, acc, nxt, logits)
    z = logits.cpu().numpy().reshape(B, k + 1, -1)
    assert (np.isnan(z).sum(-1) == 1).all()
    want = [_decide(z[b], drafts[b].tolist(), u.reshape(B, k + 1, 2)[b], top_k) for b in range(B)]
    assert list(zip(acc.cpu().tolist(), nxt.cpu().tolist())) == want


@pytest.mark.parametrize("V,top_k", [(31 * 128, 31), (31 * 128, 1), (32 * 128, 32), (32 * 128, 1), (33 * 128, 33)])
def test_sampling_fewest_blocks(V, top_k):
    """Around 32 blocks, from which on the block maxima narrow a row."""
    exact, report, _ = _case(V, 6, 3, 1.0, top_k, 2.0, seed=V + top_k)
    assert exact + len(report) == 6 and len(report) <= 1, report

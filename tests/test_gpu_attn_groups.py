"""Attention with one, two and four key groups per query block against float64: lists
of every length around the group count, ragged last chunks, entries outside the
layer, and rows whose mass sits in one group only. (Rows that leave the reference-0 form:
test_gpu_attn_references.)"""
import numpy as np
import pytest

from launch_rules import attn_groups

pytestmark = pytest.mark.gpu


def reference(q, k, v, count, idx, bq, bk, scale):
    """softmax over the listed blocks' tokens (duplicates count twice), float64."""
    import torch

    H, N, _ = q.shape
    out = torch.zeros(H, N, 64, dtype=torch.float64)
    for h in range(H):
        for i in range(count.shape[1]):
            keys = [torch.arange(j * bk, min((j + 1) * bk, N)) for j in idx[h, i, :int(count[h, i])].tolist()
                    if 0 <= j < idx.shape[2]]
            if not keys:
                continue
            t = torch.cat(keys)
            s = q[h, i * bq:(i + 1) * bq].double() @ k[h, t].double().T * scale
            out[h, i * bq:(i + 1) * bq] = torch.softmax(s, 1) @ v[h, t].double()
    return out


CASES = [(1, 70 * 64 - 5, 64, 64, 4), (2, 33 * 128 + 1, 128, 128, 4), (2, 40 * 128 - 64, 128, 128, 4), (3, 700, 64, 64, 2),
         (3, 1100, 128, 128, 2), (2, 1025, 64, 128, 2), (2, 900, 128, 64, 2), (70, 45 * 64 + 3, 64, 64, 1),
         # both sides of the rule's lines: 7 chunks, 512 rows with 31 and 32, 63 and 64 chunks
         (1, 6 * 64, 64, 64, 1), (1, 7 * 64 - 9, 64, 64, 2), (18, 31 * 64 - 7, 64, 64, 1), (18, 32 * 64 - 7, 64, 64, 2),
         (17, 63 * 64, 128, 64, 1), (17, 64 * 64 - 1, 128, 128, 2)]


@pytest.mark.parametrize("spread", [1.0, 30.0])
@pytest.mark.parametrize("H,N,bq,bk,G", CASES)
def test_groups(H, N, bq, bk, G, spread):
    import torch

    import paper_2609_35593_amd as ress

    n_qb, n_kb = -(-N // bq), -(-N // bk)
    assert attn_groups(H, n_qb, n_kb, bq, bk) == G
    rng = np.random.default_rng(H * 1000 + N)
    gen = torch.Generator().manual_seed(N + int(spread))
    q, k, v = (torch.randn(H, N, 64, generator=gen) for _ in range(3))
    # Keys of every third block point along (or, spread > 1, far along and against) one direction of the queries,
    # so that a row's mass differs from group to group.
    d = torch.randn(64, generator=gen)
    d /= d.norm()
    q += 2.0 * d
    for j in range(n_kb):
        k[:, j * bk:(j + 1) * bk] += (spread if j % 3 == 0 else -spread if j % 3 == 1 else 0.0) * d
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    count = torch.zeros(H, n_qb, dtype=torch.int32)
    idx = torch.full((H, n_qb, n_kb), -1, dtype=torch.int32)
    for h in range(min(H, 3)):
        for i in range(n_qb):
            c = i % 8 if i < n_qb - 1 else n_kb  # empty rows, one block, ... and a full list
            c = min(c, n_kb)
            pick = np.sort(rng.choice(n_kb, c, replace=False)).astype(np.int32)
            if c and i % 3 == 2:
                pick[-1] = n_kb - 1  # the ragged last block
            if c > 2 and i % 5 == 4:
                pick[rng.integers(c)] = n_kb + 7  # contributes nothing
            if c > 2 and i % 8 == 3:
                pick[:] = np.where(np.arange(c) < c - 1, -1, pick)  # one entry that counts, after others that do not
            count[h, i] = c
            idx[h, i, :c] = torch.from_numpy(pick)
    hs = min(H, 3)
    got = ress.ress_sparse_attn_out_f32(q.cuda(), k.cuda(), v.cuda(), count.cuda(), idx.cuda(), bq=bq, bk=bk).cpu().double()
    ref = reference(q[:hs], k[:hs], v[:hs], count[:hs], idx[:hs], bq, bk, 0.125)
    assert torch.isfinite(got).all()
    assert torch.all(got[hs:] == 0.0)
    err = (got[:hs] - ref).abs()
    # The probabilities are rounded to bf16 (2^-9 each, and their sum with them) and, in the reference-0 form, so is
    # the scaled Q: 2^-9 of every product in a logit, at most 2^-9 L with L the largest sum of |q_d k_d| / 8. A weight
    # that is off by a factor 1 + e moves the output by at most 2 e max|v|.
    L = float((q[:hs].double().abs() @ k[:hs].double().abs().transpose(1, 2)).max()) * 0.125
    bound = 2.0 * (2.0 ** -8 + 2.0 ** -9 * L) * float(v.double().abs().max())
    assert float(err.max()) <= bound and float(err.mean()) <= 2e-3, (float(err.max()), bound, float(err.mean()))


@pytest.mark.parametrize("N,G", [(512, 2), (4096, 4)])
def test_groups_share_one_form_of_the_scores(N, G):
    """A row's first 64 keys choose between pre-scaled and exact scores for all of its groups: the other chunks' logits
    are large, equal in two chunks of different groups and opposite in V, so the output is the difference of the two
    groups' weights (0, but up to 0.1 where one group's scores are pre-scaled and the other's are not)."""
    import torch

    import paper_2609_35593_amd as ress

    assert attn_groups(1, N // 128, N // 64, 128, 64) == G
    q, k, v = (torch.zeros(1, N, 64) for _ in range(3))
    q[0, :, 0] = torch.linspace(50.0, 60.0, N)  # base-2 logits of 90 to 108 against 10, about 1 against 0.1
    k[0, :, 0] = 0.1
    for chunk, sign in ((1, 1.0), (G, -1.0)):  # the second group's first chunk, the first group's second
        k[0, 64 * chunk:64 * chunk + 64, 0] = 10.0
        v[0, 64 * chunk:64 * chunk + 64] = sign
    out = ress.ress_dense_attn(*(t.to(torch.bfloat16).cuda() for t in (q, k, v)), bq=128, bk=64).float().cpu()
    # Equal scores, so equal weights: what is left is the rounding of the output and keys 2^-80 of the mass.
    assert float(out.abs().max()) <= 2.0 ** -9, float(out.abs().max())


@pytest.mark.parametrize("H,N", [(12, 1500), (256, 300)])
def test_counts_beyond_the_layer(H, N):
    """Counts outside [0, n_kb] are clamped wherever they are read: by the rows and by the order of the work, which
    adds them up over the heads."""
    import torch

    import paper_2609_35593_amd as ress

    gen = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn(H, N, 64, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    n_qb, n_kb = -(-N // 128), -(-N // 64)
    idx = torch.arange(n_kb, dtype=torch.int32, device="cuda").expand(H, n_qb, n_kb).contiguous()
    raw = torch.full((H, n_qb), 2 ** 31 - 1, dtype=torch.int32, device="cuda")
    raw[1::3] = 3
    raw[2::5] = -2 ** 31
    out = [ress.ress_sparse_attn(q, k, v, c, idx, bq=128, bk=64) for c in (raw, raw.clamp(0, n_kb))]
    assert torch.equal(*out)
    assert torch.equal(out[0][0], ress.ress_dense_attn(q, k, v, bq=128, bk=64)[0])

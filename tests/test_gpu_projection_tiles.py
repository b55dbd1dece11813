"""The projections over layouts of full (256-row) and half (128-row) tiles: half tiles
alone, full tiles alone, and full tiles finished by half ones, at tile edges and one
token off them, against float64 products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def tiles(T, n):
    """(full, half) row tiles of T tokens and n column tiles: the library's rule, restated."""
    m = -(-T // 256)
    whole = m * n // 256
    mf = whole * 256 // n
    mh = -(-(T - mf * 256) // 128)
    half_rounds = max(0, mh * n - (whole * 256 - mf * n) + 255) // 256
    return (mf, mh) if 10 * whole + 6 * half_rounds < 10 * -(-m * n // 256) else (m, 0)


def check(got, ref, mag, K):
    """Nearest bf16 of a float32 sum: half a step of the result, and the sum's own error."""
    bound = np.abs(ref) * 2.0 ** -8 + K * 2.0 ** -24 * mag + 1e-30
    assert np.all(np.abs(got - ref) <= bound), float((np.abs(got - ref) / bound).max())


# (tokens, heads, kind of layout of the QKV projection)
QKV = [(1, 4, "half"), (127, 4, "half"), (128, 4, "half"), (129, 4, "half"), (257, 4, "half"), (3000, 16, "full"),
       (22016 + 1, 4, "mixed"), (22016 + 129, 4, "mixed"), (22016 + 300, 4, "mixed")]


@pytest.mark.parametrize("bq,bk", [(128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("T,H,kind", QKV)
def test_qkv_tiles(T, H, kind, bq, bk):
    import torch

    import paper_2609_35593_amd as ress

    mf, mh = tiles(T, 3 * H * 64 // 256)
    assert kind == ("mixed" if mf and mh else "half" if mh else "full")
    dm = 64 * H
    gen = torch.Generator(device="cuda").manual_seed(T + bq + bk)
    x = torch.randn(T, dm, generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn(3 * dm, dm, generator=gen, device="cuda") * dm ** -0.5).to(torch.bfloat16)
    gram = torch.randn(H, 64, 64, generator=gen, device="cuda")
    out = ress.ress_qkv_proj_pool(x, w, gram, bq=bq, bk=bk)
    rows = torch.unique(torch.tensor([0, T // 2, T - 1] + [t for t in range(max(0, T - 300), T)], device="cuda"))
    ref = (x[rows].double() @ w.double().T).view(-1, 3, H, 64)
    mag = (x[rows].double().abs() @ w.double().abs().T).view(-1, 3, H, 64)
    for i, n in enumerate("qkv"):
        check(out[n][:, rows].double().transpose(0, 1).cpu().numpy(), ref[:, i].cpu().numpy(), mag[:, i].cpu().numpy(), dm)
    # The pooled state is the one the selection pools from the same outputs.
    n_kb = -(-T // bk)
    budget = np.full(H, min(n_kb, max(2, n_kb // 3)), np.int32)
    kw = dict(bq=bq, bk=bk, want_debug=True)
    a = ress.ress_select(out["q"], out["k"], out["v"], gram, budget, workspace=out["workspace"],
                         pooled_in_workspace=True, **kw)
    b = ress.ress_select(out["q"], out["k"], out["v"], gram, budget, **kw)
    for n in ("kept_count", "kept_idx", "drift", "key", "prob"):
        assert torch.equal(a[n], b[n]), n


OUT = [(1, 4, "half"), (128, 4, "half"), (255, 4, "half"), (9000, 16, "full"), (64 * 256 + 1, 16, "mixed"),
       (64 * 256 + 200, 16, "mixed")]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("T,H,kind", OUT)
def test_out_tiles(T, H, kind, f32):
    import torch

    import paper_2609_35593_amd as ress

    mf, mh = tiles(T, H * 64 // 256)
    assert kind == ("mixed" if mf and mh else "half" if mh else "full")
    dm = 64 * H
    gen = torch.Generator(device="cuda").manual_seed(T + f32)
    o = torch.randn(H, T, 64, generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn(dm, dm, generator=gen, device="cuda") * dm ** -0.5).to(torch.bfloat16)
    r = torch.randn(T, dm, generator=gen, device="cuda").to(torch.float32 if f32 else torch.bfloat16)
    cat = o.permute(1, 0, 2).reshape(T, dm)
    ref = (r.double() + cat.double() @ w.double().T).cpu().numpy()
    mag = (r.double().abs() + cat.double().abs() @ w.double().abs().T).cpu().numpy()
    f = ress.ress_out_proj_residual_f32 if f32 else ress.ress_out_proj_residual
    got = f(o, w, r)
    assert torch.equal(got, f(o, w, r, resid_out=r))  # in place
    got = got.double().cpu().numpy()
    if f32:
        assert np.all(np.abs(got - ref) <= (dm + 1) * 2.0 ** -24 * mag)
    else:
        check(got, ref, mag, dm)

"""bf16, d = 128: the scoring sweeps' forms that are chosen by the length of a key split and by the number of KV groups.  Against
the sums in 64 bits, on KV groups spread over the launch (the first and the last among them)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# keys per split: 768 / groups splits (at least two from 16 chunks of 128 keys on), in whole chunks
@pytest.mark.parametrize("L,Hkv,g,m,tau", [
    (1, 1, 2, 2049, 20),             # splits of one chunk
    (64, 8, 1, 4096, 32),            # 512 groups, two splits: one full round of four blocks of 64 keys per CU in sweep 2
    (64, 8, 3, 4097, 32),            # 2176 keys per split
    (64, 8, 4, 4200, 7),             # the last split ends in the middle of a chunk
    (128, 6, 1, 1000, 33),           # 768 groups, one split: chunks of 128 keys in sweep 2
    (128, 6, 3, 2200, 32),           # two splits, 1536 blocks: one round of sweep 1's blocks of 32 keys
    (128, 8, 2, 2200, 32),           # 2048 blocks: of 64 keys for up to three row blocks
    (128, 8, 3, 2201, 31),
    (128, 8, 4, 2200, 32),           # four
    (127, 6, 1, 2200, 64),           # 762 groups
    (96, 8, 8, 16500, 64),           # 16 row blocks, 8320 keys per split: sweep 1's long form
    (96, 8, 5, 16300, 57),           # 8192
])
def test_sweep_forms(L, Hkv, g, m, tau):
    import paper_2410_23317_amd as V
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    d, p = 128, 0.01
    shape = V.make_shape(1, L, Hkv * g, Hkv, d, m, tau, "bf16")
    new = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    k, q = new(1, L, Hkv, m, d), new(1, L, Hkv * g, tau, d)
    scores = torch.full((1, L, Hkv, m), float("nan"), device="cuda")
    row_max = torch.full((1, L, Hkv * g, tau), float("nan"), device="cuda")
    row_sum = torch.full_like(row_max, float("nan"))
    nnz = torch.full((1, L, Hkv * g), -1, dtype=torch.int64, device="cuda")
    ws = torch.empty(V.vlc_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    V.vlc_score(shape, q, k, None, p, scores, row_max, row_sum, nnz, ws)
    again, nnz2 = torch.full_like(scores, float("nan")), torch.full_like(nnz, -1)
    V.vlc_score_from_stats(shape, q, k, None, p, row_max, row_sum, again, nnz2)
    torch.cuda.synchronize()
    assert torch.allclose(scores, again, rtol=5e-5, atol=1e-7)
    groups = L * Hkv
    see = torch.arange(m, device="cuda") <= torch.arange(m - tau, m, device="cuda")[:, None]      # causal
    for x in sorted({0, 1, groups // 3, groups // 2, groups - 2, groups - 1} & set(range(groups))):
        l, h = divmod(x, Hkv)
        s = q[0, l, h * g:(h + 1) * g].double() @ k[0, l, h].double().T.contiguous() * d ** -0.5
        s = torch.where(see, s, float("-inf"))
        M = s.max(-1).values
        Z = torch.exp(s - M[..., None]).sum(-1)
        torch.testing.assert_close(row_max[0, l, h * g:(h + 1) * g].double(), M, rtol=1e-5, atol=1e-5)
        torch.testing.assert_close(row_sum[0, l, h * g:(h + 1) * g].double(), Z, rtol=5e-5, atol=1e-7)
        want = (torch.exp(s - M[..., None]) / Z[..., None]).sum((0, 1))
        torch.testing.assert_close(scores[0, l, h].double(), want, rtol=5e-5, atol=1e-7)
        margin = s - M[..., None] - torch.log(torch.tensor(p, dtype=torch.float64))
        count, near = (margin >= 0).sum((1, 2)), (margin.abs() < 1e-5 * s.abs().clamp(1)).sum((1, 2))
        for n in (nnz, nnz2):
            assert bool(((n[0, l, h * g:(h + 1) * g] - count).abs() <= near).all()), (l, h)

"""Launches over a layer range whose upper bound of block-units is far beyond what the chip holds at once: a capped grid whose blocks
take several units each.  Against attention in 64 bits over the rows that the cache itself holds."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,g,fp8", [("bf16", 64, 1, False), ("bf16", 128, 4, False), ("bf16", 64, 3, True), ("bf16", 128, 7, True), ("f32", 64, 2, False), ("f32", 128, 8, False)])
@pytest.mark.parametrize("merge", [1, 2], ids=["in-kernel", "merge-kernel"])
def test_capped_grids_take_every_unit(dtype, d, g, fp8, merge):
    """128 requests of 8 KV heads, 16 layers, the first four in use: 1024 rows and a bound of nine units of each, 9216 blocks for 1024 to 3000
    units of 27 slots in the mean (in fp32 with d = 128 28 MB, which could hide 5700 blocks), against a cap of 768 blocks (256
    CUs).  Three appends, one layer at a time, then ranges of two."""
    import paper_2410_23317_amd as V
    from paper_2410_23317_amd.pipeline import VLCachePath, cache_layer_view
    B, L, Hkv, m, T, LU = 128, 16, 8, 1024, 4, 4
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + g)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda").to(dt)
    path = VLCachePath(V.make_shape(B, L, Hkv * g, Hkv, d, m, 16, dtype), alpha=(1, 64), T_max=T,
                       options=V.make_options(layer_unit_slots=128, kv_fp8=int(fp8), decode_merge=merge))
    r = np.random.default_rng(g)
    share = r.random((B, L)) ** 6 + 1e-3
    kk = np.maximum(1, np.floor(share / share.sum(1, keepdims=True) * 400)).astype(np.int32)     # at most 415 per request, of 432
    kk[:3] = 1
    kk[:3, :4] = [[390, 3, 1, 1], [1, 128, 127, 129], [127, 1, 250, 2]]
    path.scores.copy_(torch.rand(path.scores.shape, generator=gen, device="cuda"))
    path.topk_compact(new(B, L, Hkv, m, d), new(B, L, Hkv, m, d), k=torch.from_numpy(kk).cuda())
    path.status()
    tol = dict(rtol=1e-2, atol=2e-2) if dtype == "bf16" else dict(rtol=1e-4, atol=1e-4)
    for t in range(T):
        q, kn, vn = new(LU, B, Hkv * g, d), new(LU, B, Hkv, d), new(LU, B, Hkv, d)
        out = torch.full_like(q, float("nan"))
        for l0, l1 in [(l, l + 1) for l in range(LU)] if t < T - 1 else [(0, 2), (2, 4)]:
            path.decode(l0, l1, q[l0:l1], kn[l0:l1], vn[l0:l1], None, out[l0:l1])
        path.status()
        for b in range(B):
            for l in range(LU):
                k, v, idx = cache_layer_view(path.cache, b, l, appended=t + 1)
                if fp8:
                    k, v = (x[0].view(torch.float8_e4m3fn).double() * x[1].double()[..., None] for x in (k, v))
                k, v = k.double(), v.double()
                s = (q[l, b].double().view(Hkv, g, 1, d) * k[:, None]).sum(-1) * d ** -0.5
                want = (torch.softmax(s, -1)[..., None] * v[:, None]).sum(2).view(Hkv * g, d)
                torch.testing.assert_close(out[l, b].double(), want, msg=lambda m_: f"step {t} b={b} l={l}: {m_}", **tol)
                assert int(idx[:, -1].min()) == int(idx[:, -1].max()) == m + t

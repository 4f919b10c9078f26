"""Decode on values at the ends of their types: logits of -inf (a masked key: infinite entries, or products that overflow), NaN
keys, infinite values.  Against attention in 64 bits over the rows that the cache itself holds."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import assert_close, make_shape, out_tol
from oracle import vlcache_oracle as O

pytestmark = pytest.mark.gpu

ROWS = [1, 30, 31, 32, 33, 63, 64, 127, 128, 129, 300, 500, 1290]
PER_LAYER = [False, True]


def _setup(dtype, d, g, fp8, T, mask=None, fill=None):
    """One layer per entry of ROWS; q[..., 0] is 1, so that entry 0 of a key alone decides whether its logit is infinite.
    mask: kept positions (every one of a row's leading `mask` kept positions) whose keys hold -inf there."""
    import paper_2410_23317_amd as V
    from paper_2410_23317_amd.pipeline import VLCachePath
    cfg = W.custom_config(cid=81, name="values", dtype=dtype, d=d, Hq=2 * g, Hkv=2, m=1400, tau=16, lead_text=9, n_visual=1300,
                          L=len(ROWS), B=1, sinks=6, alphas=((1, 5),))
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    r = np.random.default_rng(d + g)
    put = lambda x: torch.from_numpy(x.astype(np.float32)).to(dt).cuda()
    k, v = r.standard_normal((1, cfg.L, 2, cfg.m, d)), r.standard_normal((1, cfg.L, 2, cfg.m, d))
    if mask:
        k[:, :, :, mask[0]:mask[1], 0] = -np.inf
    q = r.standard_normal((T, cfg.L, 1, cfg.Hq, d))
    q[..., 0] = 1.0
    kn, vn = r.standard_normal((T, cfg.L, 1, 2, d)), r.standard_normal((T, cfg.L, 1, 2, d))
    path = VLCachePath(make_shape(cfg), alpha=(1, 1), T_max=T,
                       options=V.make_options(unit_slots=128, layer_unit_slots=128, kv_fp8=int(fp8)))
    if fill is not None:
        path.cache.arena.fill_(fill)                 # bytes that the compaction does not write keep this value
    path.scores.copy_(torch.arange(cfg.m, 0, -1, device="cuda").float().expand(path.scores.shape))       # the leading positions are kept
    path.topk_compact(put(k), put(v), k=torch.tensor([ROWS], dtype=torch.int32, device="cuda"))
    path.status()
    return cfg, path, put, q, kn, vn


def _rows(path, l, appended):
    from paper_2410_23317_amd.pipeline import cache_layer_view
    k, v, _ = cache_layer_view(path.cache, 0, l, appended=appended)
    if path.cache.layout.kv_fp8:
        deq = lambda x: x[0].view(torch.float8_e4m3fn).double() * x[1].double()[..., None]
        return deq(k).cpu().numpy(), deq(v).cpu().numpy()
    return k.double().cpu().numpy(), v.double().cpu().numpy()


def _decode(cfg, path, put, q, kn, vn, t, per_layer):
    out = torch.empty((cfg.L, 1, cfg.Hq, cfg.d), dtype=torch.float32 if cfg.dtype == "f32" else torch.bfloat16, device="cuda")
    dq, dk, dv = put(q[t]), put(kn[t]), put(vn[t])
    for l0, l1 in [(l, l + 1) for l in range(cfg.L)] if per_layer else [(0, cfg.L)]:
        path.decode(l0, l1, dq[l0:l1], dk[l0:l1], dv[l0:l1], None, out[l0:l1])
    torch.cuda.synchronize()
    return dq.double().cpu().numpy(), out.double().cpu().numpy()


@pytest.mark.parametrize("per_layer", PER_LAYER, ids=["all-layers", "per-layer"])
@pytest.mark.parametrize("masked", ["inf", "overflow"])
@pytest.mark.parametrize("dtype,d,g,fp8", [("bf16", 128, 4, False), ("bf16", 64, 3, False), ("bf16", 128, 7, True), ("bf16", 64, 2, True),
                                           ("f32", 64, 2, False), ("f32", 128, 5, False)])
def test_an_appended_row_of_logit_minus_infinity_weighs_nothing(dtype, d, g, fp8, masked, per_layer):
    """Step 0 appends a row whose logit is -inf for every head, step 1 an ordinary one."""
    cfg, path, put, q, kn, vn = _setup(dtype, d, g, fp8, T=2)
    if masked == "inf":
        kn[0, ..., 0] = -np.inf
    else:                                            # finite keys, infinite products
        q[0, ..., 0] = 2.0 ** 100
        q[0, ..., 1:] = 0
        kn[0] = 0
        kn[0, ..., 0] = -3e38
    for t in range(2):
        dq, out = _decode(cfg, path, put, q, kn, vn, t, per_layer)
        for l in range(cfg.L):
            k, v = _rows(path, l, appended=t + 1)
            k, v = np.delete(k, ROWS[l], 1), np.delete(v, ROWS[l], 1)           # the masked row
            assert_close(out[l, 0], O.decode_attn(dq[l, 0], k, v, cfg.d ** -0.5), what=f"step {t} row of {ROWS[l]}", **out_tol(cfg))
    path.status()


@pytest.mark.parametrize("per_layer", PER_LAYER, ids=["all-layers", "per-layer"])
@pytest.mark.parametrize("lo,hi", [(0, 20), (0, 32), (32, 64), (5, 130), (0, 256)])
@pytest.mark.parametrize("dtype,d,g", [("bf16", 128, 4), ("bf16", 64, 1), ("f32", 64, 3)])
def test_kept_rows_of_logit_minus_infinity_weigh_nothing(dtype, d, g, lo, hi, per_layer):
    """Positions lo to hi of the prompt are masked by infinite keys: parts of tiles, whole tiles, whole units.  The first step's
    appended row keeps every softmax defined."""
    cfg, path, put, q, kn, vn = _setup(dtype, d, g, False, T=1, mask=(lo, hi))
    dq, out = _decode(cfg, path, put, q, kn, vn, 0, per_layer)
    for l in range(cfg.L):
        k, v = _rows(path, l, appended=1)
        live = np.isfinite(k[0, :, 0])
        assert_close(out[l, 0], O.decode_attn(dq[l, 0], k[:, live], v[:, live], cfg.d ** -0.5), what=f"row of {ROWS[l]}", **out_tol(cfg))


@pytest.mark.parametrize("dtype,d,g,fp8", [("bf16", 128, 4, False), ("bf16", 64, 3, False), ("f32", 64, 2, False)])
def test_infinite_values_and_nan_keys_stay_where_they_belong(dtype, d, g, fp8):
    """KV head 0's appended row holds an infinite value element (that output element is infinite, the others are not touched),
    KV head 1's a NaN key (every output of its heads is NaN)."""
    cfg, path, put, q, kn, vn = _setup(dtype, d, g, fp8, T=2)
    for t in range(2):
        if t == 0:
            vn[0, :, :, 0, 5] = np.inf
            kn[0, :, :, 1, 3] = np.nan
        dq, out = _decode(cfg, path, put, q, kn, vn, t, per_layer=bool(t))
        for l in range(cfg.L):
            k, v = _rows(path, l, appended=t + 1)
            assert np.isinf(out[l, 0, :g, 5]).all() and np.isnan(out[l, 0, g:]).all(), (t, ROWS[l])
            v = np.where(np.isinf(v), 0, v)
            want = O.decode_attn(dq[l, 0, :g], k[:1], v[:1], cfg.d ** -0.5)
            rest = np.arange(d) != 5
            assert_close(out[l, 0, :g][:, rest], want[:, rest], what=f"step {t} row of {ROWS[l]}", **out_tol(cfg))


@pytest.mark.parametrize("dtype,fp8,d,g", [("f32", False, d, g) for d in (64, 128) for g in range(1, 9)] +
                         [("bf16", fp8, d, g) for fp8 in (False, True) for d in (64, 128) for g in (4, 7)])
def test_rows_around_the_edges_of_tiles_and_units(dtype, fp8, d, g):
    """Rows that end before, on and behind a 32-slot tile and a 128-slot unit, of 1 to 11 units, grown by three appends; all bytes of
    the arena are NaN beforehand, so that what a cache does not hold shows if a tile lets it through."""
    cfg, path, put, q, kn, vn = _setup(dtype, d, g, fp8, T=3, fill=255)
    for t in range(3):
        dq, out = _decode(cfg, path, put, q, kn, vn, t, per_layer=t != 1)
        for l in range(cfg.L):
            k, v = _rows(path, l, appended=t + 1)
            assert_close(out[l, 0], O.decode_attn(dq[l, 0], k, v, cfg.d ** -0.5), what=f"step {t} row of {ROWS[l]}", **out_tol(cfg))
            if not fp8:                              # the appended row, bit for bit
                assert np.array_equal(k[:, -1], put(kn[t, l, 0]).double().cpu().numpy()) and np.array_equal(v[:, -1], put(vn[t, l, 0]).double().cpu().numpy())
    path.status()


@pytest.mark.parametrize("merge", [1, 2], ids=["in-kernel", "merge-kernel"])
@pytest.mark.parametrize("d,g", [(64, 1), (64, 4), (128, 2), (128, 7)])
def test_fp32_outputs_are_the_rounded_quotient(d, g, merge):
    """A query of zeros: every probability is 1, the sums are whole numbers below 2^24 and exact, so the output has to be their
    quotient to the last bit; rows of one unit, of two to eight, and of more."""
    import paper_2410_23317_amd as V
    from paper_2410_23317_amd.pipeline import VLCachePath
    rows = [1, 7, 100, 129, 300, 500, 900, 1023, 1025, 1200, 1290]
    cfg = W.custom_config(cid=82, name="quotient", dtype="f32", d=d, Hq=2 * g, Hkv=2, m=1400, tau=16, lead_text=9, n_visual=1300,
                          L=len(rows), B=1, sinks=6, alphas=((1, 5),))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(g)
    k = torch.randn((1, cfg.L, 2, cfg.m, d), generator=gen, device="cuda")
    v = torch.randint(-8000, 8001, (1, cfg.L, 2, cfg.m, d), generator=gen, device="cuda").float()
    vn = torch.randint(-8000, 8001, (cfg.L, 1, 2, d), generator=gen, device="cuda").float()
    path = VLCachePath(make_shape(cfg), alpha=(1, 1), T_max=2,
                       options=V.make_options(unit_slots=128, layer_unit_slots=128, decode_merge=merge))
    path.scores.copy_(torch.arange(cfg.m, 0, -1, device="cuda").float().expand(path.scores.shape))
    path.topk_compact(k, v, k=torch.tensor([rows], dtype=torch.int32, device="cuda"))
    q = torch.zeros((cfg.L, 1, cfg.Hq, d), device="cuda")
    out = torch.empty_like(q)
    for l0, l1 in [(0, cfg.L)] + [(l, l + 1) for l in range(cfg.L)]:
        appends = l0 == 0 and l1 == cfg.L                           # then once more per layer, over the same rows
        path.decode(l0, l1, q[l0:l1], k[0, l0:l1, :, 0].unsqueeze(1).contiguous() if appends else None, vn[l0:l1] if appends else None, None, out[l0:l1])
        torch.cuda.synchronize()
        for l in range(l0, l1):
            _, vals = _rows(path, l, appended=1)
            want = (vals.sum(1).astype(np.float32) / np.float32(rows[l] + 1)).astype(np.float32)
            got = out[l, 0].cpu().numpy().reshape(2, g, d)
            assert np.array_equal(got, np.repeat(want[:, None], g, 1)), (l0, l1, rows[l], int((got != want[:, None]).sum()))
    path.status()

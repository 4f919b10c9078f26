"""The append count of a cache: every wave of every block of a decode launch reads it, the block that holds the last ticket
writes the new one.  A model of that protocol, all interleavings of it, on the CPU; and launches whose blocks mostly hold
units reserved for later appends (their tickets are the earliest) on the GPU."""
import numpy as np
import pytest
import torch

WAVES = 3


def _reads(units_of_block, barrier):
    """All counts that a wave can meet, over every interleaving of a launch whose block i holds units_of_block[i] units.
    A wave reads the count, passes the block's barrier (if there is one), and wave 0 then takes a ticket per unit; the one
    that takes the launch's last ticket publishes count 1."""
    n_units = sum(units_of_block)
    met = set()
    start = (tuple((0,) * WAVES for _ in units_of_block), 0, 0)     # program counters per wave; tickets taken; the count
    seen, todo = {start}, [start]
    while todo:
        pcs, tickets, count = todo.pop()
        for b, block in enumerate(pcs):
            for w, pc in enumerate(block):
                tk, ct = tickets, count
                if pc == 0:                                          # the read
                    met.add(count)
                elif pc == 1:                                        # the barrier: until every wave of the block is behind its read
                    if barrier and min(block) < 1:
                        continue
                elif w == 0 and pc - 2 < units_of_block[b]:          # a ticket
                    tk += 1
                    if tk == n_units:
                        ct = 1
                else:
                    continue
                new = list(pcs)
                new[b] = block[:w] + (pc + 1,) + block[w + 1:]
                state = (tuple(new), tk, ct)
                if state not in seen:
                    seen.add(state)
                    todo.append(state)
    return met


@pytest.mark.parametrize("units_of_block", [(1,), (1, 1), (1, 1, 1), (2, 1), (3, 2)])
def test_no_wave_meets_the_new_count(units_of_block):
    assert _reads(units_of_block, barrier=True) == {0}
    assert _reads(units_of_block, barrier=False) == {0, 1}           # the model does see what the barrier is there for


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16-cache", "fp8-cache"])
@pytest.mark.parametrize("per_layer", [False, True], ids=["all-layers", "per-layer"])
def test_appends_of_launches_full_of_reserved_units(per_layer, fp8):
    """Rows of 1 to 200 slots and 1024 reserved ones in units of 128: seven of eight blocks have nothing to read.  After 60
    steps every row holds each step's position once, in order, and (bf16 cache) its rows bit for bit."""
    import paper_2410_23317_amd as V
    from paper_2410_23317_amd.pipeline import VLCachePath, cache_layer_view
    B, L, Hkv, g, d, m, T = 3, 4, 8, 2, 128, 400, 60
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    path = VLCachePath(V.make_shape(B, L, Hkv * g, Hkv, d, m, 16, "bf16"), alpha=(1, 2), T_max=1024,
                       options=V.make_options(unit_slots=128, layer_unit_slots=128, kv_fp8=int(fp8)))
    kk = np.random.default_rng(6).integers(1, 201, (B, L)).astype(np.int32)
    path.scores.copy_(torch.rand(path.scores.shape, generator=gen, device="cuda"))
    path.topk_compact(new(B, L, Hkv, m, d), new(B, L, Hkv, m, d), k=torch.from_numpy(kk).cuda())
    q, kn, vn = new(T, L, B, Hkv * g, d), new(T, L, B, Hkv, d), new(T, L, B, Hkv, d)
    out = torch.empty_like(q)
    for t in range(T):
        for l0, l1 in [(l, l + 1) for l in range(L)] if per_layer else [(0, L)]:
            path.decode(l0, l1, q[t, l0:l1], kn[t, l0:l1], vn[t, l0:l1], None, out[t, l0:l1])
    path.status()
    assert bool(torch.isfinite(out.float()).all())
    for b in range(B):
        for l in range(L):
            k, v, idx = cache_layer_view(path.cache, b, l, appended=T)
            k0 = int(kk[b, l])
            for h in range(Hkv):
                assert idx[h][k0:].cpu().tolist() == [m + t for t in range(T)], (b, l, h)
                if not fp8:
                    assert torch.equal(k[h][k0:], kn[:, l, b, h]) and torch.equal(v[h][k0:], vn[:, l, b, h]), (b, l, h)

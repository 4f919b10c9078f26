"""The scoring sweeps at the sizes where their division of the work can go wrong: bf16 with d = 64 and fp32 storage on the
matrix cores (score_wave.hip), ragged batches of bf16 with d = 128 (score_mfma.hip), and the plain-ALU sweeps of every storage
type and head dimension (score_simple.hip).  One key, one window row, remainders of the 32-key tiles and 32-row blocks, each
block form (up to 4, 8, 16 row blocks, blocks shared between heads), windows that take several launches, waves that walk
several tiles, ragged batches with NaN in all padding; each by vlc_score and from the statistics it wrote.  Against the
oracle, to the tolerances of the scoring path (fp32 accumulation of products that are exact in fp32, respectively rounded
once; a 1-ulp exponential)."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import SCORE_TOL, assert_close, check_nnz, torch_dtype
from oracle import vlcache_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,Hq,Hkv,lens", [
    ("bf16", 64, 2, 2, [(1, 1)]),                                # one key
    ("bf16", 64, 4, 1, [(31, 1), (33, 33)]),                     # shorter than a tile; the window is the whole prompt
    ("bf16", 64, 8, 2, [(2049, 32)]),                            # 4 row blocks, 9 splits, the last with a tile of one key
    ("bf16", 64, 5, 1, [(300, 32), (257, 7)]),                   # 5 row blocks
    ("bf16", 64, 8, 1, [(515, 33), (515, 5)]),                   # 16 row blocks; 8 for the shorter window
    ("bf16", 64, 8, 1, [(700, 65), (64, 64), (40, 3)]),          # 24 row blocks: two launches, the second empty for the others
    ("f32", 64, 4, 2, [(544, 32), (512, 31)]),
    ("f32", 64, 7, 1, [(385, 40)]),                              # 14 row blocks: the 16-wave form
    ("f32", 64, 3, 1, [(1000, 200), (95, 95)]),                  # 21 row blocks: two launches
    ("f32", 128, 4, 2, [(1, 1), (290, 29)]),
    ("f32", 128, 6, 2, [(333, 64), (65, 1)]),                    # 6 row blocks of 512-byte rows
    ("f32", 128, 6, 1, [(2200, 50)]),                            # 12: two launches
    ("bf16", 64, 8, 1, [(300, 1)]),                              # windows of up to 16 rows: eight heads' rows in one block
    ("bf16", 64, 7, 1, [(513, 3), (77, 2)]),                     # heads padded to four rows, the second request's too
    ("bf16", 64, 5, 1, [(64, 16), (16, 16)]),                    # two heads per block, the third block half empty
    ("f32", 64, 8, 1, [(290, 16), (65, 9)]),                     # four blocks
    ("f32", 64, 6, 2, [(100, 5)]),                               # heads padded to eight rows, a block and a half
    ("f32", 64, 2, 1, [(300, 1), (77, 1)]),                      # two rows of fp32: the plain-ALU sweeps
    ("f32", 128, 1, 1, [(257, 2)]),
    ("f32", 64, 3, 1, [(300, 1)]),                               # three: the matrix cores
    ("f32", 128, 8, 1, [(130, 9), (40, 1)]),
    ("f32", 128, 3, 1, [(70, 17)]),                              # one row more: a block per head
    # 8 KV groups of long prompts: splits of 24 tiles (of 32 for the 16-wave form), two or three tiles per wave, the last ones short
    ("bf16", 64, 4, 4, [(20001, 20)]),
    ("bf16", 64, 20, 4, [(20001, 64)]),                          # 10 row blocks
    ("bf16", 64, 4, 2, [(20001, 20), (9000, 3)]),                # the second request ends in the middle of the splits
    ("bf16", 64, 4, 4, [(20001, 5)]),                            # shared row blocks
    ("f32", 64, 8, 4, [(20001, 33)]),
    ("f32", 64, 12, 4, [(17000, 70)]),                           # the 16-wave form
    ("f32", 128, 4, 4, [(17000, 40)]),
    ("f32", 128, 4, 4, [(17000, 3)]),
    ("bf16", 128, 4, 1, [(600, 100), (500, 64), (257, 20)]),     # 16, 8 and 4 row blocks in one launch
    ("bf16", 128, 8, 1, [(700, 70), (300, 33), (65, 5)]),        # 24, 16 and 8: the first needs a second launch
])
def test_sweeps_match_the_oracle(dtype, d, Hq, Hkv, lens):
    _check_sweeps(dtype, d, Hq, Hkv, lens)


@pytest.mark.parametrize("Hq,lens", [
    (4, [(300, 8), (300, 9), (290, 16), (133, 17), (300, 24), (300, 25), (64, 1)]),      # one to four groups of eight rows in the only block of a head
    (3, [(400, 33), (400, 40), (390, 41), (257, 56), (400, 57), (33, 33)]),              # the same in its second block, heads packed across blocks
    (7, [(300, 50), (280, 63)]),                                                         # 11 packed blocks, 14 padded
    (8, [(420, 90), (300, 89)]),                                                         # 23 packed blocks in two launches, 24 padded
    (1, [(200, 100), (101, 97)]),
])
def test_window_rows_that_do_not_fill_their_blocks(Hq, lens):
    """bf16, d = 128: sweep 1 packs the heads' rows, sweep 2 leaves out groups of eight rows that are all padding."""
    _check_sweeps("bf16", 128, Hq, 1, lens)


@pytest.mark.parametrize("dtype,d,Hq,Hkv,lens", [
    ("bf16", 64, 4, 1, [(31, 1), (33, 33)]),
    ("bf16", 64, 14, 2, [(600, 50)]),
    ("bf16", 128, 8, 2, [(700, 70), (300, 33), (65, 5)]),
    ("f32", 64, 2, 1, [(800, 600)]),                             # 19 stages of 32 window rows
    ("f32", 64, 4, 2, [(300, 20), (123, 9), (511, 31)]),
    ("f32", 128, 6, 2, [(333, 64), (65, 1)]),
    ("f32", 128, 3, 1, [(1, 1)]),
])
def test_plain_alu_sweeps_match_the_oracle(dtype, d, Hq, Hkv, lens):
    """The sweeps that VLC_SHAPE_SCORE_PLAIN_ALU asks for, in each of their four instances."""
    import paper_2410_23317_amd as V
    _check_sweeps(dtype, d, Hq, Hkv, lens, V.VLC_SHAPE_SCORE_PLAIN_ALU)


def _check_sweeps(dtype, d, Hq, Hkv, lens, flags=0):
    import paper_2410_23317_amd as V
    B, L = len(lens), 2
    m, tau = max(x[0] for x in lens), max(x[1] for x in lens)
    cfgs = [W.custom_config(cid=800 + b, name=f"wave-{b}", dtype=dtype, d=d, Hq=Hq, Hkv=Hkv, m=mb, tau=tb, lead_text=0,
                            n_visual=mb, L=L, B=1, sinks=min(4, mb), alphas=((1, 5),)) for b, (mb, tb) in enumerate(lens)]
    dt = torch_dtype(cfgs[0])
    q_win = torch.full((B, L, Hq, tau, d), float("nan"), dtype=dt, device="cuda")
    k = torch.full((B, L, Hkv, m, d), float("nan"), dtype=dt, device="cuda")
    host = {}
    for b, cfg in enumerate(cfgs):
        for l in range(L):
            t = host[b, l] = W.layer_inputs(cfg, 0, l)
            q_win[b, l, :, : cfg.tau].copy_(torch.from_numpy(t["q_win"]).to(dt))
            k[b, l, :, : cfg.m].copy_(torch.from_numpy(t["k"]).to(dt))
    lens_t = torch.tensor(lens, dtype=torch.int32, device="cuda") if B > 1 else None
    scales = W.sm_scale(cfgs[0])
    shape = V.make_shape(B, L, Hq, Hkv, d, m, tau, dtype, lens=lens_t, flags=flags)
    ws = torch.full((V.vlc_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    scores, row_max, row_sum = new(B, L, Hkv, m), new(B, L, Hq, tau), new(B, L, Hq, tau)
    nnz = torch.full((B, L, Hq), 77, dtype=torch.int64, device="cuda")
    sm = torch.from_numpy(scales).cuda()
    V.vlc_score(shape, q_win, k, sm, 0.01, scores, row_max, row_sum, nnz, ws)
    again, nnz2 = new(B, L, Hkv, m), torch.full_like(nnz, 77)
    V.vlc_score_from_stats(shape, q_win, k, sm, 0.01, row_max, row_sum, again, nnz2)
    torch.cuda.synchronize()
    for b, cfg in enumerate(cfgs):
        assert torch.all(torch.isnan(row_max[b, :, :, cfg.tau:])), "window rows beyond the request's are left untouched"
        for l in range(L):
            t = host[b, l]
            psi, _, M, Z = O.score(t["q_win"], t["k"], scales[l])
            assert_close(row_max[b, l, :, : cfg.tau].cpu().numpy(), M, atol=2e-5, rtol=2e-6, what=f"b={b} l={l} row_max")
            assert_close(row_sum[b, l, :, : cfg.tau].cpu().numpy(), Z, atol=0, rtol=5e-5, what=f"b={b} l={l} row_sum")
            for got, counts, what in ((scores, nnz, f"b={b} l={l}"), (again, nnz2, f"b={b} l={l} from statistics")):
                assert torch.all(got[b, l, :, cfg.m:] == 0), "keys beyond the request's prompt score zero"
                assert_close(got[b, l, :, : cfg.m].cpu().numpy(), psi, what=what + " scores", **SCORE_TOL)
                check_nnz(counts[b, l].cpu().numpy(), t["q_win"], t["k"], scales[l], 0.01, what + " nnz")


def _upload(dtype, d, L, Hq, Hkv, m, tau, cid):
    """One request on the GPU (q_win [1,L,Hq,tau,d], k, v [1,L,Hkv,m,d]) and the host arrays of its layers."""
    cfg = W.custom_config(cid=cid, name=f"wave-{cid}", dtype=dtype, d=d, Hq=Hq, Hkv=Hkv, m=m, tau=tau, lead_text=0, n_visual=m,
                          L=L, B=1, sinks=4, alphas=((1, 5),))
    dt = torch_dtype(cfg)
    host = [W.layer_inputs(cfg, 0, l) for l in range(L)]
    dev = [torch.from_numpy(np.stack([t[n] for t in host])[None]).to(dt).cuda() for n in ("q_win", "k", "v")]
    return host, dev, W.sm_scale(cfg)


def _score(V, q_win, k, sm, dtype, flags=0, stats=None):
    """vlc_score (or, with stats = (row_max, row_sum), vlc_score_from_stats): scores, row_max, row_sum, counts."""
    (B, L, Hq, tau, d), (Hkv, m) = q_win.shape, k.shape[2:4]
    shape = V.make_shape(B, L, Hq, Hkv, d, m, tau, dtype, flags=flags)
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    scores, nnz = new(B, L, Hkv, m), torch.full((B, L, Hq), 77, dtype=torch.int64, device="cuda")
    row_max, row_sum = stats or (new(B, L, Hq, tau), new(B, L, Hq, tau))
    if stats:
        V.vlc_score_from_stats(shape, q_win, k, sm, 0.01, row_max, row_sum, scores, nnz)
    else:
        ws = torch.full((V.vlc_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
        V.vlc_score(shape, q_win, k, sm, 0.01, scores, row_max, row_sum, nnz, ws)
    torch.cuda.synchronize()
    return scores, row_max, row_sum, nnz


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128), ("bf16", 128)])
@pytest.mark.parametrize("plain", [False, True])
def test_a_layers_logit_scale_may_be_zero_or_negative(dtype, d, plain):
    """The scale is any finite number: zero makes every softmax uniform over the keys a row may see, a negative one
    turns the order of the logits around.  The causal mask holds either way."""
    import paper_2410_23317_amd as V
    host, (q, k, _), _ = _upload(dtype, d, 4, 4, 2, 300, 21, 820)
    scales = np.array([0.0, -0.09, 0.09, -0.0], dtype=np.float32)
    scores, row_max, row_sum, nnz = _score(V, q, k, torch.from_numpy(scales).cuda(), dtype, int(plain) * V.VLC_SHAPE_SCORE_PLAIN_ALU)
    for l, t in enumerate(host):
        what = f"scale {scales[l]}"
        psi, _, M, Z = O.score(t["q_win"], t["k"], scales[l])
        assert_close(scores[0, l].cpu().numpy(), psi, what=what + " scores", **SCORE_TOL)
        assert_close(row_max[0, l].cpu().numpy(), M, atol=2e-5, rtol=2e-6, what=what + " row_max")
        assert_close(row_sum[0, l].cpu().numpy(), Z, atol=0, rtol=5e-5, what=what + " row_sum")
        check_nnz(nnz[0, l].cpu().numpy(), t["q_win"], t["k"], scales[l], 0.01, what + " nnz")


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("plain", [False, True])
def test_keys_with_infinite_entries_score_zero(dtype, d, plain):
    """Keys that every window row gives a logit of -inf (a caller's way to mask them) have weight 0 and disturb no other
    key, also where window rows are padded to whole row blocks."""
    import paper_2410_23317_amd as V
    host, (q, k, _), scales = _upload(dtype, d, 2, 4, 2, 300, 21, 821)
    gone = [0, 5, 31, 32, 190, 277]                     # the last key that every row sees is 279
    q[..., 0] = 1.0
    k[:, :, :, gone, 0] = float("-inf")
    scores, row_max, row_sum, nnz = _score(V, q, k, torch.from_numpy(scales).cuda(), dtype, int(plain) * V.VLC_SHAPE_SCORE_PLAIN_ALU)
    for l in range(2):
        what = f"l={l}"
        qh, kh = q[0, l].float().cpu().numpy(), k[0, l].float().cpu().numpy()
        psi, _, M, Z = O.score(qh, kh, scales[l])
        assert np.all(psi[:, gone] == 0)
        assert_close(scores[0, l].cpu().numpy(), psi, what=what + " scores", **SCORE_TOL)
        assert_close(row_max[0, l].cpu().numpy(), M, atol=2e-5, rtol=2e-6, what=what + " row_max")
        assert_close(row_sum[0, l].cpu().numpy(), Z, atol=0, rtol=5e-5, what=what + " row_sum")
        nnz_o, *_ = O.sparsity(qh, kh, scales[l], 0.01)
        assert np.abs(nnz[0, l].cpu().numpy() - nnz_o).sum() <= 2       # a threshold decision within rounding


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
def test_scores_from_the_calls_own_statistics_are_as_accurate_as_its_scores(dtype, d):
    """vlc_score_from_stats on the row maxima and sums that vlc_score wrote.  A row's maximum is rounded to fp32, which at
    logits of a few hundred shifts every exponent by 1e-5; the row sum belongs to the rounded value, so the shift
    cancels and the two calls agree to the rounding of an exponential and a sum (a few times 2^-24 per term, 6e-8)."""
    import paper_2410_23317_amd as V
    _, (q, k, _), _ = _upload(dtype, d, 2, 4, 2, 1500, 33, 822)
    sm = torch.tensor([3.1, 0.7], device="cuda")        # logits of up to about 500
    scores, row_max, row_sum, _ = _score(V, q, k, sm, dtype)
    again = _score(V, q, k, sm, dtype, stats=(row_max, row_sum))[0]
    want = scores.double()
    assert ((again.double() - want).norm() / want.norm()).item() < 3e-7


@pytest.mark.parametrize("L", [1, 32])
def test_ragged_windows_on_both_sides_of_the_launch_per_class(L):
    """bf16, d = 128, windows of 12, 8, 4 and 8 row blocks in one batch: with 32 KV groups (one launch for all) and with
    1024 (requests of up to 8 row blocks in a launch of their own), by vlc_score and from its statistics.  NaN in the padding."""
    import paper_2410_23317_amd as V
    lens, Hq, Hkv, d, m, tau = [(1030, 70), (700, 33), (129, 20), (90, 64)], 32, 8, 128, 1030, 70
    B = len(lens)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    q = torch.randn((B, L, Hq, tau, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    k = torch.randn((B, L, Hkv, m, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    for b, (mb, tb) in enumerate(lens):
        q[b, :, :, tb:] = float("nan")
        k[b, :, :, mb:] = float("nan")
    lens_t = torch.tensor(lens, dtype=torch.int32, device="cuda")
    shape = V.make_shape(B, L, Hq, Hkv, d, m, tau, "bf16", lens=lens_t)
    ws = torch.full((V.vlc_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    scores, row_max, row_sum = new(B, L, Hkv, m), new(B, L, Hq, tau), new(B, L, Hq, tau)
    nnz = torch.full((B, L, Hq), 77, dtype=torch.int64, device="cuda")
    V.vlc_score(shape, q, k, None, 0.01, scores, row_max, row_sum, nnz, ws)
    again, nnz2 = new(B, L, Hkv, m), torch.full_like(nnz, 77)
    V.vlc_score_from_stats(shape, q, k, None, 0.01, row_max, row_sum, again, nnz2)
    torch.cuda.synchronize()
    for b, (mb, tb) in enumerate(lens):
        for got in (scores, again):
            assert torch.all(got[b, :, :, mb:] == 0), "keys beyond the request's prompt score zero"
            np.testing.assert_allclose(got[b].sum(-1).cpu().numpy(), Hq // Hkv * tb, rtol=1e-4)
        assert torch.all(torch.isnan(row_max[b, :, :, tb:])), "window rows beyond the request's are left untouched"
        for l in (0, L - 1):
            qh, kh = q[b, l, :, :tb].float().cpu().numpy(), k[b, l, :, :mb].float().cpu().numpy()
            psi, _, M, Z = O.score(qh, kh, d ** -0.5)
            for got, cnt, what in ((scores, nnz, f"b={b} l={l}"), (again, nnz2, f"b={b} l={l} from statistics")):
                assert_close(got[b, l, :, :mb].cpu().numpy(), psi, what=what + " scores", **SCORE_TOL)
                check_nnz(cnt[b, l].cpu().numpy(), qh, kh, d ** -0.5, 0.01, what + " nnz")
            assert_close(row_max[b, l, :, :tb].cpu().numpy(), M, atol=2e-5, rtol=2e-6, what=f"b={b} l={l} row_max")
            assert_close(row_sum[b, l, :, :tb].cpu().numpy(), Z, atol=0, rtol=5e-5, what=f"b={b} l={l} row_sum")


@pytest.mark.parametrize("dtype,d,Hq,lens", [
    ("bf16", 64, 4, [(8300, 7)]),                       # 33 splits of 8 tiles, shared row blocks
    ("f32", 64, 1, [(16500, 33)]),                      # 65 splits: a second round of the merging wave's lanes
    ("f32", 128, 2, [(9000, 20), (500, 3)]),            # the shorter request has no key in most splits
])
def test_few_groups_of_long_prompts_are_merged_by_a_kernel_of_their_own(dtype, d, Hq, lens):
    """Fewer than 8 KV groups and more than 32 x 256 keys: more key splits than the column sweep merges itself.  Scores,
    statistics and counts against the oracle, and the counts of the standalone sparsity sweep."""
    import paper_2410_23317_amd as V
    _check_sweeps(dtype, d, Hq, 1, lens)
    m, tau = lens[0]
    _, (q, k, _), scales = _upload(dtype, d, 2, Hq, 1, m, tau, 823)
    sm = torch.from_numpy(scales).cuda()
    nnz = _score(V, q, k, sm, dtype)[3]
    shape = V.make_shape(1, 2, Hq, 1, d, m, tau, dtype)
    alone = torch.full_like(nnz, 77)
    ws = torch.full((V.vlc_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")
    V.vlc_sparsity(shape, q, k, sm, None, 0.01, alone, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(alone, nnz)


@pytest.mark.parametrize("L,d,Hq,m,tau,plain", [(2, 64, 2, 300, 1, True), (2, 128, 1, 257, 2, True), (2, 64, 3, 300, 1, False),
                                                (2, 64, 1, 2048, 2, True), (2, 64, 1, 2049, 2, False),
                                                (64, 128, 1, 2048, 1, True), (65, 128, 1, 2048, 1, False)])
def test_one_or_two_rows_of_fp32_take_the_plain_alu_sweeps(L, d, Hq, m, tau, plain):
    """Which kernels run, told by their rounding: the bits of the flagged call or not (up to two rows, 2048 keys, 64 MiB of K)."""
    import paper_2410_23317_amd as V
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    q = torch.randn((1, L, Hq, tau, d), generator=gen, device="cuda")
    k = torch.randn((1, L, 1, m, d), generator=gen, device="cuda")
    got = _score(V, q, k, None, "f32")
    flagged = _score(V, q, k, None, "f32", V.VLC_SHAPE_SCORE_PLAIN_ALU)
    assert all(torch.equal(a, b) for a, b in zip(got, flagged)) == plain
    stats = _score(V, q, k, None, "f32", stats=got[1:3])[0]
    np.testing.assert_allclose(stats.cpu().numpy(), flagged[0].cpu().numpy(), rtol=5e-5, atol=1e-7)
    np.testing.assert_allclose(got[0].cpu().numpy(), flagged[0].cpu().numpy(), rtol=5e-5, atol=1e-7)

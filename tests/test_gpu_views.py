"""GPU parity of the views update (Sec. 2.2; App. A.2, Eq. 10-11): window
ring, bookkeeping and boundary states bit-exact, summary (eta, m) against the
oracle's incremental fp64 merge."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import Pair, check_views

pytestmark = pytest.mark.gpu

# bf16 with grouped query heads (4 q heads per kv head), two layers
MINI_BF16 = synth.QWEN3_8B.replace(name="mini-bf16", hidden=512, n_q_heads=8, n_kv_heads=2,
                                   mlp=1024, vocab=5003, n_layers=2, n_feat_layers=3,
                                   window=64)


@pytest.mark.parametrize("shape,gscale", [(synth.TINY, 1.0), (synth.TINY, 8.0),
                                          (MINI_BF16, 1.0), (MINI_BF16, 8.0)])
def test_prefill_then_decode(gpu_lib, shape, gscale):
    G = synth.make_G(shape, scale=gscale, device="cuda")
    p = Pair(gpu_lib, shape, 3, G)
    p.prefill(700, 256, ragged=5)          # ragged last chunk, n > W in one update
    check_views(p)
    p.decode(40, shape.block + 1, np.random.default_rng(0))   # includes n = 0 updates
    check_views(p)


def test_short_prefix_partial_window(gpu_lib):
    s = synth.TINY
    p = Pair(gpu_lib, s, 2, synth.make_G(s, device="cuda"))
    p.prefill(9, 9)
    check_views(p)
    p.decode(3, 2, np.random.default_rng(1))
    check_views(p)


def test_empty_update_is_bit_identical(gpu_lib):
    s = MINI_BF16
    p = Pair(gpu_lib, s, 2, synth.make_G(s, device="cuda"))
    p.prefill(100, 100)
    torch.cuda.synchronize()
    before = p.views.arena.clone()
    pos = p.views.pos.clone()
    K, V, h = synth.decode_rows(s, 2, s.block + 1, 0, device="cuda")
    p.views.update(torch.zeros(2, dtype=torch.int32, device="cuda"), K, V, h)
    torch.cuda.synchronize()
    assert torch.equal(before, p.views.arena)
    assert torch.equal(pos, p.views.pos)


def test_out_of_range_count_sets_sticky_flag(gpu_lib):
    s = synth.TINY
    p = Pair(gpu_lib, s, 3, synth.make_G(s, device="cuda"))
    p.prefill(50, 50)
    torch.cuda.synchronize()
    before = p.views.arena.view(3, -1).clone()
    K, V, h = synth.decode_rows(s, 3, 4, 0, device="cuda")
    n = torch.tensor([2, 5, -1], dtype=torch.int32, device="cuda")   # 5 > max_new = 4; -1 < 0
    p.views.update(n, K, V, h)
    assert p.views.status() == gpu_lib.LDR_ERANGE
    after = p.views.arena.view(3, -1)
    assert torch.equal(before[1], after[1]) and torch.equal(before[2], after[2])
    assert not torch.equal(before[0], after[0])
    assert p.views.pos.cpu().tolist() == [52, 50, 50]
    assert p.views.status(clear=True) == gpu_lib.LDR_ERANGE
    assert p.views.status() == gpu_lib.LDR_OK


# query tiles of 2, 4 and 8 waves at both head widths; rows around the edges of
# a 32-row tile and of the window, row ranges over several workgroups (one or
# two sequences: 256 rows split in two, 1000 in seven or so), ragged and empty
# counts, every update continuing from the one before
@pytest.mark.parametrize("hq,d,drop", [(8, 128, 0), (4, 128, 0), (16, 64, 0), (8, 64, 0),
                                       (8, 128, 1), (8, 128, 2), (8, 64, 6)])
def test_row_tiles_and_ranges(gpu_lib, hq, d, drop):
    s = MINI_BF16.replace(n_q_heads=hq, head_dim=d, drop_views=drop)
    p = Pair(gpu_lib, s, 2, None if drop & 2 else synth.make_G(s, device="cuda"))
    for i, (a, b) in enumerate([(1, 0), (31, 33), (32, 1), (0, 65), (255, 256), (1000, 129),
                                (97, 1000), (17, 3)]):
        K, V, h = synth.decode_rows(s, 2, max(a, b) + (i & 1), i, device="cuda")
        p.ingest([a, b], K, V, h)
        # P enters as two bf16 terms, within 2^-17 of itself: |dM| <= 2^-17
        # sum p |v|, and a weighted mean of |v| over N(0, 1) rows stays below
        # the largest |M| or 1
        check_views(p, atol_m=2.0 ** -17)
    assert p.views.status() == 0


# more than 512 workgroups of (group, layer, sequence): two tiles without a loader
@pytest.mark.parametrize("hq,d,drop", [(8, 128, 0), (4, 128, 0), (8, 64, 0), (8, 64, 2)])
def test_two_tiles_of_many_sequences(gpu_lib, hq, d, drop):
    """33 to 64 rows: ragged and empty second tiles, a window they wrap."""
    batch = 150
    s = MINI_BF16.replace(n_q_heads=hq, head_dim=d, drop_views=drop)
    p = Pair(gpu_lib, s, batch, None if drop & 2 else synth.make_G(s, device="cuda"),
             oracle_seqs=[0, 1, 2, batch - 1])
    for i, (n, less) in enumerate([(33, 1), (64, 31), (48, 40)]):
        K, V, h = synth.decode_rows(s, batch, n, i, device="cuda")
        p.ingest([n - b % 3 * less if n > b % 3 * less else 0 for b in range(batch)], K, V, h)
        check_views(p, atol_m=2.0 ** -17)   # as test_row_tiles_and_ranges


def test_long_update_without_a_workspace(gpu_lib):
    """One workgroup per (group, layer, sequence) walks all rows: the same copies,
    and the summary to fp32 sums in another order."""
    s = MINI_BF16
    G = synth.make_G(s, device="cuda")
    a, b = (Pair(gpu_lib, s, 2, G) for _ in range(2))
    L = gpu_lib.lib()
    for i, n in enumerate([(1000, 300), (513, 1000)]):
        K, V, h = synth.decode_rows(s, 2, 1000, i, device="cuda")
        nt = torch.tensor(n, dtype=torch.int32, device="cuda")
        a.ingest(n, K, V, h)
        ptr = [t.data_ptr() for t in (nt, K, V, h)]
        st = torch.cuda.current_stream().cuda_stream
        ws = torch.empty(64, dtype=torch.uint8, device="cuda")
        for w, sz in ((ws.data_ptr(), 64), (ws.data_ptr() + 8, 1 << 40)):   # short; misaligned
            assert L.ldr_views_update_ws(b.views.handle, ptr[0], 1000, *ptr[1:], w, sz,
                                         st) == gpu_lib.LDR_EINVAL
        assert L.ldr_views_update(b.views.handle, ptr[0], 1000, *ptr[1:], st) == 0
        check_views(a, atol_m=2.0 ** -17)
        b.ost = a.ost
        check_views(b, atol_m=2.0 ** -17)   # as test_row_tiles_and_ranges


def test_long_updates_on_a_stream_of_their_own(gpu_lib):
    """The workspace belongs to the handle's stream; a long first prefix."""
    s = MINI_BF16
    G = synth.make_G(s, device="cuda")
    a = Pair(gpu_lib, s, 2, G)
    rows = [synth.decode_rows(s, 2, 1000, i, device="cuda") for i in range(2)]
    n = torch.tensor([1000, 700], dtype=torch.int32, device="cuda")
    for K, V, h in rows:
        a.ingest([1000, 700], K, V, h)
    check_views(a, atol_m=2.0 ** -17)
    v = gpu_lib.Views(s, 2, G, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    v.init(n, *rows[0])
    v.update(n, *rows[1])
    torch.cuda.synchronize()
    assert torch.equal(v.pos, a.views.pos)
    for x, y in zip((*v.window(), *v.summary()), (*a.views.window(), *a.views.summary())):
        assert torch.equal(x, y)


def test_handles_hold_no_workspace(gpu_lib):
    """A handle's own device memory is its status block, whatever its shape."""
    vs = [gpu_lib.Views(synth.QWEN3_8B, 1, synth.make_G(synth.QWEN3_8B, device="cuda"))
          for _ in range(16)]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for v in vs:
        v.init()
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] <= 16 * (2 << 20)   # pages of 2 MB at most


def test_infinite_value_and_nan_key(gpu_lib):
    """An infinite value in the last, ragged tile leaves the summary of its
    group's heads not finite in that dimension only (infinite, or NaN where the
    two bf16 terms of its probability differ in sign; padding rows add
    nothing), a NaN key makes the summary of its group's heads NaN and leaves
    the others alone; split and unsplit rows."""
    s = MINI_BF16
    for rows in (20, 300):
        v = gpu_lib.Views(s, 1, synth.make_G(s, device="cuda")).init()
        K, V, h = synth.decode_rows(s, 1, rows, 3, device="cuda")
        V[0, rows - 1, 0, 0, 5] = float("inf")
        K[0, rows - 2, 1, 1, 7] = float("nan")
        v.update(torch.tensor([rows], dtype=torch.int32, device="cuda"), K, V, h)
        M, eta = (x[0].cpu() for x in v.summary())
        rep = s.n_q_heads // s.n_kv_heads
        fin = torch.isfinite(M[0])
        assert not fin[:rep, :, 5].any()
        fin[:rep, :, 5] = True
        assert fin.all() and torch.isfinite(eta[0]).all()
        assert torch.isnan(M[1, rep:]).all() and torch.isnan(eta[1, rep:]).all()
        assert torch.isfinite(M[1, :rep]).all() and torch.isfinite(eta[1, :rep]).all()


@pytest.mark.slow
def test_full_size_qwen3_8b_prefill_sampled(gpu_lib):
    """Qwen3-8B shape, batch 16, prefix 32768 ingested in 4096-row chunks, then
    64 decode updates of 17 rows: bookkeeping for all sequences, window and
    summary of two sampled sequences against the oracle."""
    s = synth.QWEN3_8B
    G = synth.make_G(s, device="cuda")
    p = Pair(gpu_lib, s, 16, G, oracle_seqs=[0, 13])
    p.prefill(32768, 4096)
    rng = np.random.default_rng(2)
    for st in range(64):
        K, V, h = synth.decode_rows(s, 16, 17, st, device="cuda")
        p.ingest([17] * 16, K, V, h)
    del rng
    assert p.views.pos.cpu().tolist() == [32768 + 64 * 17] * 16
    check_views(p)

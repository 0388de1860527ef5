"""Decode attention where its pipeline steps and its merge can go wrong: units whose pages do not
fill their last step of one, two or four tiles, ranges longer than the 64 steps described at a time,
units cut into many pieces, and bad pages or scales next to a step's live tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_15930_amd import inputs, sl
from parity import assert_parity, oracle_full

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]
DEV = "cuda:0"
KINDS = [(64, "bf16"), (128, "bf16"), (64, "e4m3"), (128, "e4m3")]


def _say(*a):
    print(*a, flush=True)


@pytest.mark.parametrize("workers", [1, 2, 3, 11])
@pytest.mark.parametrize("D,kv", KINDS)
def test_step_and_chunk_edges(D, kv, workers):
    """1 .. 9 pages with a full, a single and a 15-token last page, and ranges of 63 .. 130 steps."""
    L = [16 * n + r for n in range(9) for r in (1, 15, 16)] + [16 * 62 + 5, 16 * 129, 16 * 257 + 1]
    _say("step edges", D, kv, workers)
    b = inputs.make_paged_batch(L, 6, 2, D, seed=D + workers, device=DEV, kv_dtype=kv)
    out = sl.run_batch(b, num_workers=workers)
    torch.cuda.synchronize()
    assert_parity(out, oracle_full(b), f"D={D} {kv} workers={workers}")


@pytest.mark.parametrize("pieces", [2, 8, 9, 16, 17, 33, 64, 65, 129])
@pytest.mark.parametrize("D,kv", KINDS)
def test_unit_cut_into_many_pieces(D, kv, pieces):
    """One KV head over `pieces` workers (a worker takes at least four tiles): the merge's first
    batch of rows, the loop after it and the second chunk of 64 weights."""
    L = [16 * 8 * pieces - 7]
    _say("pieces", D, kv, pieces)
    b = inputs.make_paged_batch(L, 7, 1, D, seed=pieces, device=DEV, kv_dtype=kv)
    out = sl.run_batch(b, num_workers=pieces)
    torch.cuda.synchronize()
    assert_parity(out, oracle_full(b), f"D={D} {kv} pieces={pieces}")


@pytest.mark.parametrize("page", [0, 1, 2, 3, 4, 6])
@pytest.mark.parametrize("D,kv", KINDS)
def test_page_outside_the_pool_at_every_place_of_a_step(D, kv, page):
    """The sequence that names it gets NaN rows, its neighbours theirs."""
    L = [100, 16 * 7, 50]
    _say("bad page", D, kv, page)
    b = inputs.make_paged_batch(L, 4, 2, D, seed=3, device=DEV, kv_dtype=kv)
    want = sl.run_batch(b, num_workers=2).clone()
    b.block_table[1, page] = b.k_pages.shape[0] if page % 2 else -1
    out = sl.run_batch(b, num_workers=2)
    torch.cuda.synchronize()
    assert torch.isnan(out[1].float()).all()
    assert torch.equal(out[0], want[0]) and torch.equal(out[2], want[2])


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 0.0])
@pytest.mark.parametrize("D", [64, 128])
def test_scales_of_pages_not_read_do_not_leak(D, bad):
    """A step's missing tiles are multiplied by no scale but those of its own pages."""
    L = [16 * n + 3 for n in range(6)]
    _say("scales", D, bad)
    b = inputs.make_paged_batch(L, 4, 2, D, seed=5, device=DEV, kv_dtype="e4m3")
    # what page 0 holds moves to a new page; page 0 and the poison page then go bad
    n = b.k_pages.shape[0]
    b.k_pages, b.v_pages = torch.cat([b.k_pages, b.k_pages[:1]]), torch.cat([b.v_pages, b.v_pages[:1]])
    b.k_scales, b.v_scales = torch.cat([b.k_scales, b.k_scales[:1]]), torch.cat([b.v_scales, b.v_scales[:1]])
    b.block_table = torch.where(b.block_table == 0, torch.full_like(b.block_table, n), b.block_table)
    want = oracle_full(b)
    for s in (b.k_scales, b.v_scales):
        s[0] = bad
        s[b.poison_page] = bad
    out = sl.run_batch(b, num_workers=3)
    torch.cuda.synchronize()
    assert_parity(out, want, f"D={D} bad={bad}")


@pytest.mark.parametrize("pages", [1, 2, 3, 5, 6, 7, 9])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_infinite_value_scale_beside_a_steps_missing_tiles(D, shared, pages):
    """Full pages of positive values, the last one with an infinite value scale: every weighted sum is
    +inf, as in the oracle, whether or not the unit's last step has tiles beyond its pages (a weight of
    zero times the scale there would make it NaN)."""
    _say("infinite scale", D, shared, pages)
    b = inputs.make_paged_batch([16 * pages] * 2, 4, 2, D, seed=pages, device=DEV, kv_dtype="e4m3")
    b.v_pages.bitwise_and_(0x3F).bitwise_or_(0x20)   # codes of 2^-3 up to 1.875
    for i in range(2):
        b.v_scales[b.block_table[i, pages - 1]] = float("inf")
    if shared:   # both sequences read the first one's pages, through the shared stream
        b.block_table[1] = b.block_table[0]
        ints = dict(dtype=torch.int32, device=DEV)
        out = sl.decode_attn_prefix_fp8(b.q, b.k_pages, b.v_pages, b.k_scales, b.v_scales, b.block_table, b.seq_lens,
                                        b.scale, torch.tensor([0, 2], **ints), torch.tensor([pages], **ints))
    else:
        out = sl.run_batch(b)
    torch.cuda.synchronize()
    assert torch.isposinf(out.float()).all()


def _append_every_slot(D, grow, B, Hkv):
    rng = np.random.default_rng(D)
    lens, N = np.arange(B, dtype=np.int32) % 33 + 1, 3 * B
    bt = rng.permutation(N).astype(np.int32).reshape(B, 3)
    gain = {"none": 1e-3, "all": 50.0, "some": np.resize([1e-3, 50.0, 1.0], Hkv)[None, :, None]}[grow]

    def row():
        x = torch.from_numpy((rng.standard_normal((B, Hkv, D)) * gain).astype(np.float32)).to(torch.bfloat16)
        return x, x.view(torch.int16).numpy().view(np.uint16)

    (k, kbits), (v, vbits) = row(), row()
    pages = [rng.integers(0, 0x7E, (N, Hkv, 16, D)).astype(np.uint8) for _ in range(2)]
    scales = [rng.uniform(0.01, 0.1, (N, Hkv)).astype(np.float32) for _ in range(2)]
    want = oracle.kv_append(kbits, vbits, bt, lens, *pages, k_scales=scales[0], v_scales=scales[1])
    got = [torch.from_numpy(a.copy()).to(DEV) for a in pages + scales]
    _say("append slots", D, grow)
    sl.kv_append(k.to(DEV), v.to(DEV), torch.from_numpy(bt).to(DEV), torch.from_numpy(lens).to(DEV), got[0], got[1],
                 k_scales=got[2], v_scales=got[3])
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy().view(np.uint8), np.ascontiguousarray(w).view(np.uint8))


@pytest.mark.parametrize("grow", ["none", "all", "some"])
@pytest.mark.parametrize("D", [64, 128])
def test_e4m3_append_at_every_slot(D, grow):
    """A tile is re-encoded by four wavefronts of four rows each: every slot, with scales that stay,
    grow, or grow in some heads, equals the oracle byte for byte; a fresh page ignores its old scale."""
    _append_every_slot(D, grow, 33, 3)


@pytest.mark.parametrize("B,Hkv", [(512, 4), (683, 3), (825, 3)])
@pytest.mark.parametrize("grow", ["none", "all", "some"])
@pytest.mark.parametrize("D", [64, 128])
def test_e4m3_append_at_every_slot_of_many_units(D, grow, B, Hkv):
    """The same around 2048 units, beyond which one wavefront re-encodes both of a unit's tiles."""
    _append_every_slot(D, grow, B, Hkv)


@pytest.mark.parametrize("D", [64, 128])
def test_e4m3_append_of_many_units_is_not_bound_by_their_old_codes(D):
    """65536 units whose scales stay: an E4M3 append stores half of a bf16 one's bytes and a scale per
    row beside them, so it stays within a few times its duration (1.4 of it on MI355X; fetching every
    unit's old codes took ten)."""
    B, H = 8192, 8
    _say("append duration", D)
    rows = [torch.ones(B, H, D, dtype=torch.bfloat16, device=DEV) for _ in "kv"]
    table = torch.arange(B, dtype=torch.int32, device=DEV)[:, None].contiguous()
    lens = torch.full((B,), 9, dtype=torch.int32, device=DEV)
    took = {}
    for kv in ("bf16", "e4m3"):
        dt = torch.bfloat16 if kv == "bf16" else torch.uint8
        pages = [torch.zeros(B, H, 16, D, dtype=dt, device=DEV) for _ in "kv"]
        kw = {} if kv == "bf16" else {n: torch.ones(B, H, device=DEV) for n in ("k_scales", "v_scales")}
        times = []
        for _ in range(12):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                sl.kv_append(*rows, table, lens, *pages, **kw)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop))
        took[kv] = sorted(times)[len(times) // 2]
    assert took["e4m3"] < 4 * took["bf16"], took


@pytest.mark.parametrize("tiles", [3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 130])
@pytest.mark.parametrize("D,kv", KINDS)
def test_worker_counts_of_small_streams(D, kv, tiles):
    """The split kernel and the merge each work out how many of the workers take part: around every
    line of that rule (four tiles per worker, for E4M3 up to half of the workers, eight beyond it),
    with units that share workers, and with shared pages."""
    lens = [16 * (tiles // 3), 16 * (tiles - 2 * (tiles // 3)) - 3, 16 * (tiles // 3) - 9]
    b = inputs.make_paged_batch(lens, 6, 2, D, seed=tiles, device=DEV, kv_dtype=kv)
    for workers in (1, 8, 9):
        _say("worker counts", D, kv, tiles, workers)
        assert_parity(sl.run_batch(b, num_workers=workers), oracle_full(b), f"{kv} tiles={tiles} workers={workers}")
    b, starts, shared = inputs.make_grpo_batch(3, 2, 16 * (tiles // 3) + 1, seed=tiles, device=DEV, num_q_heads=6,
                                               num_kv_heads=2, head_dim=D, gen_median=20.0, gen_cap=60, kv_dtype=kv)
    for workers in (8, 9):
        if kv == "e4m3":
            out = sl.decode_attn_prefix_fp8(b.q, b.k_pages, b.v_pages, b.k_scales, b.v_scales, b.block_table,
                                            b.seq_lens, b.scale, starts, shared, num_workers=workers)
        else:
            out = sl.decode_attn_prefix(b.q, b.k_pages, b.v_pages, b.block_table, b.seq_lens, b.scale, starts, shared,
                                        num_workers=workers)
        torch.cuda.synchronize()
        assert_parity(out, oracle_full(b), f"prefix {kv} tiles={tiles} workers={workers}")


def test_e4m3_append_of_the_most_units():
    """8192 sequences x 1024 heads: with two workgroups per unit more threads than a launch's first dimension holds."""
    B, H, D = 8192, 1024, 64
    _say("append units", B * H)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    rows = [torch.randn(B, H, D, generator=gen, device=DEV, dtype=torch.bfloat16) for _ in "kv"]
    pages = [torch.full((B, H, 16, D), 0xAB, dtype=torch.uint8, device=DEV) for _ in "kv"]
    scales = [torch.full((B, H), 7.0, device=DEV) for _ in "kv"]
    table = torch.arange(B, dtype=torch.int32, device=DEV)[:, None].contiguous()
    sl.kv_append(*rows, table, torch.ones(B, dtype=torch.int32, device=DEV), *pages, k_scales=scales[0],
                 v_scales=scales[1])
    torch.cuda.synchronize()
    for x, p, s in zip(rows, pages, scales):
        for i in range(0, B, 512):
            f = x[i:i + 512].float()
            a = f.abs().amax(dim=2)
            want = a / torch.full_like(a, 448.0)   # (by a Python number torch multiplies by 1/448: another rounding)
            codes = (f / want[:, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
            assert torch.equal(s[i:i + 512], want)
            assert torch.equal(p[i:i + 512, :, 0], codes)
            assert bool((p[i:i + 512, :, 1:] == 0xAB).all())


@pytest.mark.parametrize("D,kv", KINDS)
def test_prefix_sharing_with_the_most_groups(D, kv):
    """4096 sequences in 4096 groups, the most that are accepted: the kernel's arrays in LDS are at their largest."""
    B = 4096
    _say("most groups", D, kv)
    b, starts, shared = inputs.make_grpo_batch(B, 1, 20, seed=4, device=DEV, num_q_heads=2, num_kv_heads=1, head_dim=D,
                                               gen_median=10.0, gen_cap=40, kv_dtype=kv)
    assert len(starts) == B + 1 and int(shared.min()) > 0
    if kv == "e4m3":
        out = sl.decode_attn_prefix_fp8(b.q, b.k_pages, b.v_pages, b.k_scales, b.v_scales, b.block_table, b.seq_lens,
                                        b.scale, starts, shared)
    else:
        out = sl.decode_attn_prefix(b.q, b.k_pages, b.v_pages, b.block_table, b.seq_lens, b.scale, starts, shared)
    torch.cuda.synchronize()
    assert_parity(out, oracle_full(b), f"most groups D={D} {kv}")


def test_one_page_sequences_are_not_computed_as_four():
    """Thousands of sequences of one page, head_dim 64: with an E4M3 cache (steps of four tiles) a call takes about
    as long as with a bf16 one (1.01 of it on MI355X; computing the three tiles that are not there took 1.25)."""
    _say("one page")
    took = {}
    rng = np.random.default_rng(0)
    lens = rng.integers(1, 14, 5663).tolist()
    for kv in ("bf16", "e4m3"):
        b = inputs.make_paged_batch(lens, 3, 3, 64, seed=1, device=DEV, kv_dtype=kv)
        times = []
        for _ in range(15):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                sl.run_batch(b)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop))
        took[kv] = sorted(times)[len(times) // 2]
    assert took["e4m3"] < 1.13 * took["bf16"], took

"""extend_attention at the sizes where its kernels and dispatch rules change: edges of
the tiles and key steps, remainders, mixed batches.  Every row is checked against the
CPU oracle with LSE, over pools whose unused slots hold NaN."""

import numpy as np
import pytest
import torch

from gpu_harness import DEV, GpuRun, compare, oracle_rows
from paper_2609_32278_amd import kvx
from paper_2609_32278_amd import workloads as wl
from test_abi import _check_plan
from test_gpu_extend import _run_and_compare

pytestmark = pytest.mark.gpu

NAN_FILL = {wl.KV_BF16: 0x7FC0, wl.KV_FP8_E4M3: 0x7F}

# prefixes whose last key falls on each edge of a 16-slot page, of a 64-key step and of
# the four waves' round of 256 keys; one long enough for many parts
STEP_EDGES = [0, 1, 14, 15, 16, 31, 47, 48, 62, 63, 64, 65, 127, 191, 254, 255, 256, 300, 2600]


@pytest.mark.parametrize("dt", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (6, 2, 64), (16, 1, 64), (1, 1, 128)])
@pytest.mark.parametrize("split", [0, 64])
def test_decode_at_the_edges_of_pages_and_key_steps(dt, hq, hkv, d, split):
    w = wl.make_custom(STEP_EDGES, [1] * len(STEP_EDGES), hq, hkv, d, kv_dtype=dt, seed=61)
    _run_and_compare(w, f"decode_edges_{dt}_{hq}_{hkv}_{d}_{split}", want_lse=True, fill=NAN_FILL[dt],
                     split_keys=split)


# prefilling requests next to decoding ones: chunked and single-chunk decode prefixes, an
# empty prefix (one key), a request with no suffix, a prefill tile that a split of 1024 keys
# cuts into parts; enough one-token work for the mixed launch
MIXED_P = [0, 4000, 9000, 33, 15000, 700, 2047, 2048, 5000, 12345, 6000]
MIXED_E = [1, 1, 1, 130, 1, 40, 1, 1, 0, 1, 150]


def _check_mixed(w, split):
    """The batch's plan has decode units: chunks of 512 keys (2048 at most, as many as give 512
    units) or of the forced split, whose parts are numbered after the prefill tiles'."""
    items = _check_plan(w, split)
    one = w.extend_lens[items["req"]] == 1
    keys = w.num_kv_heads * int((w.prefix_lens[w.extend_lens == 1] + 1).sum())
    chunk = split or min(2048, max(512, keys // 512)) // 64 * 64
    starts = np.unique(items["key_begin"][items["req"] == 4])
    assert np.array_equal(starts, np.arange(0, 15001, chunk))
    tiles = items["part"][~one & (items["part"] >= 0)]
    chunks = items["part"][one & (items["part"] >= 0)]
    assert len(chunks) and chunks.min() == len(tiles)
    if split:
        assert 10 in items["req"][~one & (items["part"] >= 0)]


@pytest.mark.parametrize("dt", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("hq,hkv,d", [(32, 4, 128), (12, 6, 64), (64, 4, 64)])
@pytest.mark.parametrize("split,scaled_q", [(0, False), (1024, False), (0, True)])
def test_batches_that_mix_prefill_and_decode(dt, hq, hkv, d, split, scaled_q):
    w = wl.make_custom(MIXED_P, MIXED_E, hq, hkv, d, kv_dtype=dt, seed=62)
    _check_mixed(w, split)
    # decode units are always exact: compare with the exact attention at the standard gate
    _run_and_compare(w, f"mixed_{dt}_{hq}_{hkv}_{d}_{split}_{int(scaled_q)}", want_lse=True, fill=NAN_FILL[dt],
                     split_keys=split, scaled_q=scaled_q)


@pytest.mark.parametrize("dt,hq,hkv,d,split", [
    (wl.KV_BF16, 32, 4, 128, 1024), (wl.KV_FP8_E4M3, 32, 4, 128, 1024), (wl.KV_BF16, 12, 6, 64, 1024),
    (wl.KV_BF16, 32, 4, 128, 0),
    (wl.KV_BF16, 32, 4, 128, 64),  # more parts than the scratch holds of either kind: lengths are doubled
])
def test_mixed_batches_in_the_fixed_scratch(dt, hq, hkv, d, split):
    """The allocation-free call of a mixed batch: prefill and decode parts side by side in the
    scratch.  The bits of extend_attention where neither is limited, else the oracle's gate."""
    w = wl.make_custom(MIXED_P, MIXED_E, hq, hkv, d, kv_dtype=dt, seed=62)
    _check_mixed(w, split)
    print(f"[mixed] noalloc {dt} {hq}/{hkv}/{d} split {split}", flush=True)
    run = GpuRun(w, fill_bits=NAN_FILL[dt], split_keys=split)
    try:
        run.store()
        want, want_lse = run.attend(want_lse=True)
        out, lse = torch.full_like(want, float("nan")), torch.full_like(want_lse, float("nan"))
        kvx.extend_attention_noalloc(run.pool, run.batch, run.q, hq, w.sm_scale, out, lse)
        torch.cuda.synchronize()
        if split == 1024:
            assert torch.equal(out.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, want_lse)
        (ref, ref_lse), gidx = oracle_rows(w, run.q, None, want_lse=True)
        compare(out.float().cpu().numpy().astype(np.float64)[gidx], ref, f"mixed noalloc split {split}")
        assert np.abs(lse.cpu().numpy()[gidx] - ref_lse).max() <= 2e-3 * max(1.0, float(np.abs(ref_lse).max()))
    finally:
        run.close()


@pytest.mark.parametrize("dt", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("split", [0, 1024])
def test_mixed_batches_keep_nan(dt, d, split):
    """A NaN or infinity in a one-token request's query, keys or values comes out as NaN in
    just the query heads (for values: the dim) it reaches, in a mixed batch as in a tile."""
    hq, hkv = 32, 4
    P, E = [9000, 4000, 15000, 700, 12345, 2048, 8000, 33], [1, 1, 1, 40, 1, 1, 1, 130]
    w = wl.make_custom(P, E, hq, hkv, d, kv_dtype=dt, seed=65)
    kv = [wl.request_kv(w, r, DEV) for r in range(len(P))]
    q = [wl.request_q(w, r, DEV) for r in range(len(P))]
    want = torch.zeros((len(P), hq, d), dtype=torch.bool)
    q[0][0, 3] = float("nan")
    want[0, 3] = True
    q[5][0, 7, 0] = float("inf")  # infinite scores of both signs
    want[5, 7] = True
    kv[6][0][:, 2, 9] = kv[6][0][:, 2, 9].abs() + 0.125
    q[6][0, 17, 9] = float("-inf")  # no score above -inf: zeros, on an fp8 pool NaN
    want[6, 17] = dt == wl.KV_FP8_E4M3
    if dt == wl.KV_BF16:          # (storing codes clamps what is not finite)
        kv[1][0][1234, 1, 5] = float("nan")
        want[1, 8:16] = True
        kv[2][0][7777, 2, 9] = float("inf")  # NaN where the score is +inf, no weight where it is -inf
        want[2, 16:24] = (q[2][0, 16:24, 9] > 0).cpu()[:, None]
        kv[4][1][4321, 0, 11] = float("nan")
        want[4, 0:8, 11] = True
    run = GpuRun(w, overrides={"kv": lambda r: kv[r], "q": lambda r: q[r]}, split_keys=split)
    try:
        run.store()
        out = run.attend()
        for r in range(len(P)):
            rows = out[int(run.qo[r]):int(run.qo[r + 1])]
            got = torch.isnan(rows).cpu()
            assert torch.equal(got, want[r].expand_as(got)), (r, int(got.sum()), int(want[r].sum()))
        assert dt == wl.KV_FP8_E4M3 or bool((out[int(run.qo[6]), 17] == 0).all())
    finally:
        run.close()


@pytest.mark.parametrize("dt,d", [(wl.KV_BF16, 128), (wl.KV_FP8_E4M3, 128), (wl.KV_BF16, 64), (wl.KV_FP8_E4M3, 64)])
def test_decode_beyond_the_infinity_cache_gives_the_same_bits(dt, d):
    """A decode batch that reads more than 256 MB streams its pages with non-temporal
    loads: the same bits as each request by itself, at the same chunk length."""
    per = 2 * 8 * d * (2 if dt == wl.KV_BF16 else 1)  # K/V bytes per token
    n = 1 + (300 << 20) // (50000 * per)
    P = [50000 + 7 * i for i in range(n)]
    w = wl.make_custom(P, [1] * n, 32, 8, d, kv_dtype=dt, seed=63, placement="linear")
    run = GpuRun(w, split_keys=4096)
    try:
        run.store()
        whole = run.attend()
        for r in (0, n - 1):
            ids = torch.from_numpy(w.pages_of(r).copy()).to(DEV)
            one = kvx.Batch([P[r]], [1], [0, len(ids)], ids)
            out = torch.zeros_like(whole[r:r + 1])
            kvx.extend_attention(run.pool, one, run.q[r:r + 1].contiguous(), 32, w.sm_scale, out)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), whole[r:r + 1].view(torch.int16)), r
    finally:
        run.close()


@pytest.mark.parametrize("dt,d", [(wl.KV_BF16, 128), (wl.KV_FP8_E4M3, 64)])
@pytest.mark.parametrize("n,split", [(4, 0), (40, 0), (40, 4096), (256, 0), (257, 0)])
def test_decode_on_shared_prefixes_gives_the_same_bits(dt, d, n, split):
    """Requests on two shared prefixes and on pages of their own, beyond 256 MB together: in
    kernel arguments and uploaded, at the most requests whose page lists are compared and
    one more.  Every request gives the bits it gives by itself."""
    hkv, hq = 8, 16
    per = 2 * hkv * d * (2 if dt == wl.KV_BF16 else 1)  # K/V bytes per token
    shared = -(-(300 << 20) // (per * n) // 16) * 16
    tails = [1 + 37 * (r % 5) for r in range(n)]
    sp, tp = shared // 16, 12
    perm = np.random.default_rng(66).permutation(2 * sp + n * (sp + tp if n <= 40 else tp)).astype(np.int32)
    lists, at = [], 2 * sp
    for r in range(n):
        own = n <= 40 and r % 4 == 3  # a prefix of its own
        head = perm[at:at + sp] if own else perm[r % 2 * sp:(r % 2 + 1) * sp]
        at += sp if own else 0
        lists.append(np.concatenate([head, perm[at:at + tp]]))
        at += tp
    scale = np.full(hkv, 0.05, np.float32)
    pool = kvx.kv_pool_create(len(perm), 16, hkv, d, dt, *((scale, scale) if dt == wl.KV_FP8_E4M3 else ()))
    try:
        kvx.kv_pool_set_split_keys(pool, split)
        g = torch.Generator(device=DEV).manual_seed(67)
        for a in range(0, len(perm), 1024):
            ids = np.arange(a, min(a + 1024, len(perm)), dtype=np.int32)
            k, v = [torch.randn((len(ids), hkv, 16, d), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(2)]
            if dt == wl.KV_FP8_E4M3:
                k, v = [(20 * x).to(torch.float8_e4m3fn).view(torch.uint8) for x in (k, v)]
            kvx.kv_pool_write_pages(pool, ids, k.contiguous(), v.contiguous())
            torch.cuda.synchronize()
        q = torch.randn((n, hq, d), generator=g, device=DEV, dtype=torch.bfloat16)
        P = np.array([shared + t for t in tails])
        table = torch.from_numpy(np.concatenate(lists)).to(DEV)
        batch = kvx.Batch(P, [1] * n, np.arange(n + 1) * (sp + tp), table)
        assert int((P + 1).sum()) * per > 256 << 20
        whole = torch.empty_like(q)
        kvx.extend_attention(pool, batch, q, hq, d ** -0.5, whole)
        if not split:  # the chunk the batch chose
            items = kvx.extend_attention_plan(batch, hq, hkv, d)
            first = items[items["key_begin"] == 0]
            chunk = int(first["key_end"][first["part"] >= 0].max(initial=0))
            kvx.kv_pool_set_split_keys(pool, chunk)
        for r in [*range(min(n, 8)), n - 1]:
            one = kvx.Batch([P[r]], [1], [0, sp + tp], torch.from_numpy(lists[r]).to(DEV))
            out = torch.empty_like(q[r:r + 1])
            kvx.extend_attention(pool, one, q[r:r + 1].contiguous(), hq, d ** -0.5, out)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), whole[r:r + 1].view(torch.int16)), r
    finally:
        kvx.kv_pool_destroy(pool)


def test_decode_reads_a_shared_prefix_from_the_caches():
    """96 requests on one 64k prefix read it at more than twice the rate of 16 requests on pages
    of their own (2.5 times measured; 1.5 with non-temporal loads of the shared pages)."""
    hq, hkv, d, tokens = 64, 8, 128, 65536
    pages, scale = tokens // 16, np.full(hkv, 0.05, np.float32)
    pool = kvx.kv_pool_create(16 * pages + 96, 16, hkv, d, wl.KV_FP8_E4M3, scale, scale)
    try:
        us = {}
        for n, lists in ((16, [np.arange(r * pages, (r + 1) * pages) for r in range(16)]),
                         (96, [np.arange(pages)] * 96)):
            ids = np.concatenate([np.append(x, 16 * pages + r) for r, x in enumerate(lists)]).astype(np.int32)
            batch = kvx.Batch([tokens] * n, [1] * n, np.arange(n + 1) * (pages + 1), torch.from_numpy(ids).to(DEV))
            q = torch.randn((n, hq, d), device=DEV, dtype=torch.bfloat16)
            out = torch.empty_like(q)
            times = []
            for _ in range(12):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                kvx.extend_attention(pool, batch, q, hq, d ** -0.5, out)
                b.record()
                torch.cuda.synchronize()
                times.append(1000 * a.elapsed_time(b))
            us[n] = min(times)
        ratio = (96 / us[96]) / (16 / us[16])
        print(f"[shared] 16 private {us[16]:.0f} us, 96 shared {us[96]:.0f} us, rate ratio {ratio:.2f}", flush=True)
        assert ratio > 2.0
    finally:
        kvx.kv_pool_destroy(pool)


def _entries_and_tiles(items):
    """Entries of a plan in kernel arguments, one for a unit or one for eight units that differ in
    their KV head alone (all or none of the plan), and its tiles."""
    entries = len(items)
    if len(items) % 8 == 0:
        by8 = items.reshape(-1, 8)
        alike = all((by8[f] == by8[f][:, :1]).all() for f in ("req", "tok_begin", "key_begin"))
        if alike and (np.diff(by8["kv_head"], axis=1) == 1).all() and (items["req"] >= 0).all():
            entries //= 8
    return entries, len(np.unique(items[items["req"] >= 0][["req", "tok_begin"]]))


@pytest.mark.parametrize("hq,hkv,prefix,extend,split,inline", [
    (8, 8, [700, 20], [90, 300], 0, True),        # eight heads side by side: one word for eight units
    (32, 16, [700, 20, 5], [9, 40, 33], 64, True),  # two heads per XCD, split parts
    (8, 8, [8000], [200], 64, True),              # 126 parts a head
    (8, 8, [15000, 9000], [40, 300], 64, True),   # 539 words
    (8, 8, [30000, 9000], [300, 300], 64, False),  # 1252 words
    (6, 3, [300, 77, 900], [200, 300, 64], 64, True),  # a word per unit
    (4, 2, [3000, 2500], [130, 100], 64, True),   # the same, 296 words
    (4, 2, [12000, 9000], [130, 100], 64, False),  # 1064 words
    (4, 2, [20] * 130, [3] * 130, 0, False),      # unsplit: 780 words of tiles and 260 of units
    (8, 8, [20] * 130, [3] * 130, 0, True),       # 780 and 130
    (4, 2, [20] * 170, [3] * 170, 0, False),      # tiles alone are too many
    (8, 8, [5000, 300, 64], [1, 1, 1], 64, True),  # decode: entries for eight units, merges in the arguments
    (16, 8, [9000, 700], [1, 1], 64, False),      # decode: too many units
    (3, 3, [900, 31], [1, 1], 64, True),          # decode, an entry per unit
    (3, 3, [3000], [1], 64, False),               # the same, too many
])
def test_plans_in_kernel_arguments_and_uploaded(hq, hkv, prefix, extend, split, inline):
    """A decode plan of up to 110 entries and a prefill plan of up to 960 words (six for a tile, one
    for an entry) travel in the kernel arguments, larger ones are uploaded."""
    w = wl.make_custom(prefix, extend, hq, hkv, 64, seed=64)
    entries, tiles = _entries_and_tiles(_check_plan(w, split))
    assert inline == (entries <= 110 if max(extend) == 1 else 6 * tiles + entries <= 960), (entries, tiles)
    _run_and_compare(w, f"inline_{hkv}_{prefix[0]}_{extend[0]}", want_lse=True, fill=0x7FC0, split_keys=split)

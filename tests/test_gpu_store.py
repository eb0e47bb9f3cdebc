"""store_kv and raw page I/O on the GPU: pool contents bit-exact against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from gpu_harness import DEV, GpuRun
from helpers import oracle_pool_for
from paper_2609_32278_amd import kvx
from paper_2609_32278_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _case(name):
    if name == "tiny":
        return wl.make_workload("tiny")
    if name == "tiny_fp8":
        w = wl.make_workload("tiny")
        return wl.make_custom(w.prefix_lens, w.extend_lens, 4, 2, 64, kv_dtype=wl.KV_FP8_E4M3, seed=3,
                              num_pages=256)
    if name == "ragged_d128":
        return wl.make_custom([0, 5, 16, 37, 100, 3, 1000], [7, 0, 1, 29, 18, 40, 200], 8, 2, 128, seed=4)
    if name == "ragged_fp8_d128":
        return wl.make_custom([0, 5, 16, 37, 100, 3, 1000], [7, 0, 1, 29, 18, 40, 200], 8, 2, 128,
                              kv_dtype=wl.KV_FP8_E4M3, seed=5)
    # KV head counts that leave a partial pass of the store's head batches (4 per pass at
    # head_dim 128, 8 at 64)
    if name == "hkv5_d128":
        return wl.make_custom([0, 21, 300], [40, 17, 33], 10, 5, 128, seed=6)
    if name == "hkv9_fp8_d64":
        return wl.make_custom([7, 0], [50, 16], 9, 9, 64, kv_dtype=wl.KV_FP8_E4M3, seed=7)
    if name == "hkv3_d64":
        return wl.make_custom([16, 3], [64, 13], 6, 3, 64, seed=8)
    raise KeyError(name)


@pytest.mark.parametrize("name", ["tiny", "tiny_fp8", "ragged_d128", "ragged_fp8_d128", "hkv5_d128", "hkv9_fp8_d64",
                                  "hkv3_d64"])
def test_store_kv_pool_bit_exact(name):
    print(f"[store] {name}", flush=True)
    w = _case(name)
    fill = 0x5A if w.kv_dtype == wl.KV_FP8_E4M3 else 0x5A5A
    run = GpuRun(w, fill_bits=fill)
    try:
        run.store()
        torch.cuda.synchronize()
        k, v = run.read_pages(np.arange(w.num_pages, dtype=np.int32))
        t = wl.batch_tensors(w, device=DEV)
        t = {key: val.cpu() for key, val in t.items()}
        ref = oracle_pool_for(w, t, fill=fill)
        assert np.array_equal(k, ref.k), "K pool differs"
        assert np.array_equal(v, ref.v), "V pool differs"
    finally:
        run.close()


def test_write_then_read_pages_round_trip():
    print("[store] page round trip", flush=True)
    pool = kvx.kv_pool_create(40, 16, 3, 128, kvx.KVX_KV_BF16)
    try:
        ids = np.array([7, 0, 39, 12], np.int32)
        g = torch.Generator(device=DEV).manual_seed(5)
        k = torch.randint(-32768, 32767, (4, 3, 16, 128), generator=g, device=DEV, dtype=torch.int32).to(torch.int16)
        v = torch.randint(-32768, 32767, (4, 3, 16, 128), generator=g, device=DEV, dtype=torch.int32).to(torch.int16)
        kvx.kv_pool_write_pages(pool, ids, k, v)
        k2, v2 = torch.empty_like(k), torch.empty_like(v)
        kvx.kv_pool_read_pages(pool, ids, k2, v2)
        torch.cuda.synchronize()
        assert torch.equal(k, k2) and torch.equal(v, v2)
        lay = kvx.kv_pool_layout(pool)
        assert lay["v_stride_dim"] == 16 and lay["v_stride_slot"] == 1 and lay["k_stride_slot"] == 128
    finally:
        kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("scale", [1.0, 0.01, 0.0371, 0.1, 3.3e-5])
def test_fp8_store_matches_oracle_codec_for_every_bf16_value(scale):
    """All 65536 bf16 bit patterns (NaNs replaced by 0) through store_kv into an fp8
    pool: the hardware e4m3 conversion must give the oracle's codes bit for bit."""
    print(f"[store] fp8 codec scale={scale}", flush=True)
    bits = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    x = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).clone()
    x[torch.isnan(x)] = 0.0
    E, D = 512, 128
    xin = x.reshape(E, 1, D).to(DEV)
    w = wl.make_custom([0], [E], 1, 1, D, kv_dtype=wl.KV_FP8_E4M3, k_scale=[scale], v_scale=[scale],
                       placement="linear", num_pages=E // 16)
    pool = kvx.kv_pool_create(w.num_pages, 16, 1, D, kvx.KVX_KV_FP8_E4M3, w.k_scale, w.v_scale)
    try:
        ids = torch.from_numpy(w.page_ids).to(DEV)
        b = kvx.Batch(w.prefix_lens, w.extend_lens, w.page_indptr, ids)
        kvx.store_kv(pool, b, xin, xin)
        k = torch.empty((w.num_pages, 1, 16, D), dtype=torch.uint8, device=DEV)
        v = torch.empty_like(k)
        kvx.kv_pool_read_pages(pool, w.page_ids, k, v)
        torch.cuda.synchronize()
        got_k = k.cpu().numpy().reshape(-1)
        got_v = v.cpu().numpy().reshape(-1)
        inv = (1.0 / torch.tensor(scale, dtype=torch.float32))
        want = oracle.e4m3_encode((x.to(torch.float32) * inv).numpy()).reshape(-1)
        bad = np.nonzero(got_k != want)[0]
        assert len(bad) == 0, f"{len(bad)} codes differ, e.g. x={x.reshape(-1)[bad[:5]]} got {got_k[bad[:5]]} want {want[bad[:5]]}"
        assert np.array_equal(got_v, want)
    finally:
        kvx.kv_pool_destroy(pool)


def test_store_leaves_prefix_slots_of_a_shared_page_alone():
    """Suffix tokens that start mid-page must not touch the page's prefix slots."""
    print("[store] shared first page", flush=True)
    w = wl.make_custom([5, 21], [3, 40], 2, 1, 64, seed=8, num_pages=16)
    run = GpuRun(w, fill_bits=0x1234)
    try:
        before_k, before_v = run.read_pages(w.page_ids)
        run.store()
        after_k, after_v = run.read_pages(w.page_ids)
        for r in range(w.num_reqs):
            p = int(w.prefix_lens[r])
            j0 = int(w.page_indptr[r])
            page_row = j0 + p // 16
            assert np.array_equal(after_k[page_row, :, : p % 16], before_k[page_row, :, : p % 16])
            assert np.array_equal(after_v[page_row, :, : p % 16], before_v[page_row, :, : p % 16])
    finally:
        run.close()


@pytest.mark.parametrize("n", [1, 959, 960, 961, 1921, 7680, 7681])
def test_page_io_counts_around_the_argument_blocks(n):
    """Page ids travel in kernel arguments, 960 to a launch, up to 7680; more are uploaded.
    Every page must come back from where it was written."""
    print(f"[store] page io n={n}", flush=True)
    pool = kvx.kv_pool_create(n + 3, 16, 1, 64, kvx.KVX_KV_FP8_E4M3, np.ones(1, np.float32), np.ones(1, np.float32))
    try:
        g = torch.Generator(device=DEV).manual_seed(n)
        k = torch.randint(0, 127, (n, 1, 16, 64), generator=g, device=DEV, dtype=torch.uint8)
        v = torch.randint(0, 127, (n, 1, 16, 64), generator=g, device=DEV, dtype=torch.uint8)
        ids = np.random.default_rng(n).permutation(n + 3)[:n].astype(np.int32)
        kvx.kv_pool_write_pages(pool, ids, k, v)
        back = np.argsort(ids)  # read in page order: other ids per launch than at the write
        k2, v2 = torch.zeros_like(k), torch.zeros_like(v)
        kvx.kv_pool_read_pages(pool, ids[back], k2, v2)
        torch.cuda.synchronize()
        order = torch.from_numpy(back.copy()).to(DEV)
        assert torch.equal(k2, k[order]) and torch.equal(v2, v[order])
    finally:
        kvx.kv_pool_destroy(pool)

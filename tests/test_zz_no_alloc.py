"""extend_attention_noalloc (the allocation-free entry point) against extend_attention.

Two calls in a row through the C ABI, the second on a smaller batch (so it runs
on what the first left in the shared per-GPU scratch), each compared with
extend_attention on the same pool and inputs: bit for bit (both take the same
plan here, split parts included) and against the fp64 oracle with the parity
gate, also with the pool's scaled-Q setting on.  A batch whose plan does not fit the scratch is refused on the host.
"""

import numpy as np
import pytest
import torch

from gpu_harness import DEV, GpuRun, compare, oracle_rows
from paper_2609_32278_amd import kvx
from paper_2609_32278_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _both(w, split_keys=0, scaled_q=False):
    run = GpuRun(w, split_keys=split_keys, scaled_q=scaled_q)
    try:
        run.store()
        ref, ref_lse = run.attend(want_lse=True)
        out = torch.full_like(ref, float("nan"))
        lse = torch.full_like(ref_lse, float("nan"))
        kvx.extend_attention_noalloc(run.pool, run.batch, run.q, w.num_q_heads, w.sm_scale, out, lse)
        torch.cuda.synchronize()
        items = kvx.extend_attention_plan(run.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, split_keys)
        return run.q, ref, ref_lse, out, lse, items
    finally:
        run.close()


@pytest.mark.parametrize("case", ["prefill", "prefill_scaled_q", "decode"])
def test_noalloc_matches_extend_attention_on_two_calls_in_a_row(case):
    scaled_q = case == "prefill_scaled_q"  # the pool's scaled-Q setting holds for both entry points
    if case.startswith("prefill"):
        # split key ranges (partial results in the scratch), then a smaller batch
        first = wl.make_custom([4000, 129, 0, 2500], [70, 200, 300, 33], 8, 2, 128, seed=41)
        second = wl.make_custom([300, 17], [40, 9], 8, 2, 128, seed=42)
        splits = (1024, 0)
    else:
        first = wl.make_custom([9000, 3001, 64, 5000], [1, 1, 1, 1], 16, 2, 128, seed=43,
                               kv_dtype=wl.KV_FP8_E4M3)
        second = wl.make_custom([700, 20], [1, 1], 16, 2, 128, seed=44, kv_dtype=wl.KV_FP8_E4M3)
        splits = (512, 0)
    for k, (w, split) in enumerate(zip((first, second), splits)):
        print(f"[noalloc] {case} call {k}: P={w.prefix_lens.tolist()} E={w.extend_lens.tolist()} split={split}",
              flush=True)
        q, ref, ref_lse, out, lse, items = _both(w, split, scaled_q)
        parts = int((items["part"] >= 0).sum())
        if k == 0:
            assert parts > 0, "the first call should exercise the partial-result region"
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), f"{case} call {k}: outputs differ"
        assert torch.equal(lse, ref_lse), f"{case} call {k}: LSE differs"
        want, gidx = oracle_rows(w, q, None, scaled_q=scaled_q)
        got = out.float().cpu().numpy().astype(np.float64)[gidx]
        compare(got, want, f"noalloc {case} call {k}")


def test_noalloc_refuses_a_plan_larger_than_its_scratch():
    """262,400 work items of 32 B do not fit the 8 MiB plan region: refused with
    EUNSUPPORTED before any device work (buffers are whole, so even a launch would
    stay in bounds)."""
    hq = hkv = 256
    d, E = 64, 262400
    need = (E + 15) // 16
    pool = kvx.kv_pool_create(need, 16, hkv, d)
    try:
        ids = torch.arange(need, dtype=torch.int32, device=DEV)
        b = kvx.Batch([0], [E], [0, need], ids)
        items = kvx.extend_attention_plan(b, hq, hkv, d)
        assert len(items) * 32 > kvx.NOALLOC_PLAN_BYTES
        q = torch.zeros((E, hq, d), dtype=torch.bfloat16, device=DEV)
        out = torch.full_like(q, 3.0)
        with pytest.raises(kvx.KvxError) as e:
            kvx.extend_attention_noalloc(pool, b, q, hq, 0.125, out)
        assert e.value.status == kvx.KVX_EUNSUPPORTED
        assert "plan" in kvx.kvx_last_error()
        torch.cuda.synchronize()
        assert bool((out[:: 4096].float() == 3.0).all())
    finally:
        kvx.kv_pool_destroy(pool)


def test_noalloc_takes_a_batch_that_fits_only_without_padding():
    """One long request and 80000 short ones: with its XCDs evened out by padding the plan is
    larger than the scratch; the call runs it packed, to the same bits."""
    hq, hkv, d, n = 4, 2, 64, 80000
    P = np.append(100000, np.arange(n) % 30)
    E = np.append(180000, 2 + np.arange(n) % 3)
    indptr = np.concatenate([[0], np.cumsum((P + E + 15) // 16)])
    pool = kvx.kv_pool_create(int(indptr[-1]), 16, hkv, d)
    try:
        print(f"[noalloc] packed: {n + 1} requests, {indptr[-1]} pages", flush=True)
        g = torch.Generator(device=DEV).manual_seed(45)
        ids = np.arange(indptr[-1], dtype=np.int32)
        k, v = [torch.randn((len(ids), hkv, 16, d), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(2)]
        kvx.kv_pool_write_pages(pool, ids, k, v)
        b = kvx.Batch(P, E, indptr, torch.from_numpy(ids).to(DEV))
        items = kvx.extend_attention_plan(b, hq, hkv, d)
        assert len(items) * 32 > kvx.NOALLOC_PLAN_BYTES > (items["req"] >= 0).sum() * 32
        assert (items["part"] < 0).all()
        q = torch.randn((int(E.sum()), hq, d), generator=g, device=DEV, dtype=torch.bfloat16)
        want, got = torch.empty_like(q), torch.full_like(q, float("nan"))
        kvx.extend_attention(pool, b, q, hq, d ** -0.5, want)
        torch.cuda.synchronize()
        kvx.extend_attention_noalloc(pool, b, q, hq, d ** -0.5, got)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    finally:
        kvx.kv_pool_destroy(pool)

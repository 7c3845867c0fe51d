"""The allocation-free entry point cp_attn_mixed_noalloc.

It runs cp_attn_mixed's plan and kernels on the library's static device
scratch (set up once per device by cp_noalloc_init) instead of a caller
workspace.  GPU: two calls in a row through the C ABI, the second on a
smaller batch, each checked against cp_attn_mixed on the same inputs (bit for
bit: same plan, same kernels) and against the fp64 oracle.  Host: batches
whose workspace exceeds the scratch are refused before the device is
touched.
"""

import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2606_09061_amd as cp
from paper_2606_09061_amd import binding
from workloads import make_batch, make_config, make_tensors

MAX_ABS, MEAN_ABS = 2e-2, 2e-3


def _oversize_batch():
    rng = np.random.default_rng(0)
    return make_batch("big", 64, 8, 128, 16, [(32767 - i, 1) for i in range(10)], rng)


def test_noalloc_refuses_batches_beyond_its_scratch(monkeypatch):
    """Host only: the size limit is checked before any device call."""
    monkeypatch.setenv("CP_DECODE_TARGET_ITEMS", "100000")   # 256 splits per row
    b = _oversize_batch()
    d = cp.desc_for(b)
    assert cp.workspace_bytes(d, b.rows) > binding.NOALLOC_SCRATCH_BYTES
    lib = binding.load()
    r = np.ascontiguousarray(b.rows)
    fake = 1 << 20   # never dereferenced
    rc = lib.cp_attn_mixed_noalloc(ctypes.byref(d), fake, fake, fake, fake, r.ctypes.data,
                                   r.shape[0], fake, None)
    assert rc == binding.CP_ERR_WORKSPACE
    bad = np.array([[0, 10, 5, 16]], np.int32)
    assert lib.cp_attn_mixed_noalloc(ctypes.byref(d), fake, fake, fake, fake, bad.ctypes.data, 1,
                                     fake, None) == binding.CP_ERR_BAD_META
    assert lib.cp_attn_mixed_noalloc(ctypes.byref(d), None, fake, fake, fake, r.ctypes.data, 1,
                                     fake, None) == binding.CP_ERR_INVALID_ARG
    empty = np.zeros((0, 4), np.int32)
    assert lib.cp_attn_mixed_noalloc(ctypes.byref(d), None, None, None, None, empty.ctypes.data,
                                     0, None, None) == binding.CP_OK


def _two_plans_batch():
    """A chunk after 8,000 keys beside eight decode rows: cp_attn_mixed's plan
    splits the chunk further than the scratch holds; sized as for the vector
    units it fits."""
    rows = [(8000, 1000)] + [(15999, 1)] * 8
    return make_batch("two plans", 64, 8, 128, 32, rows, np.random.default_rng(4))


def test_noalloc_takes_the_plan_that_fits():
    """Host only: without a device the accepted batch fails at its first device
    call, and not for its size."""
    if torch.cuda.is_available():
        pytest.skip("stand-in addresses: for a host without a GPU")
    b = _two_plans_batch()
    d = cp.desc_for(b)
    assert cp.workspace_bytes(d, b.rows) > binding.NOALLOC_SCRATCH_BYTES
    r, fake = np.ascontiguousarray(b.rows), 1 << 20
    rc = binding.load().cp_attn_mixed_noalloc(ctypes.byref(d), fake, fake, fake, fake,
                                              r.ctypes.data, r.shape[0], fake, None)
    assert rc == binding.CP_ERR_HIP


def _run_both(batch, seed):
    """Appends with cp_kv_append, then cp_attn_mixed (caller workspace) and
    cp_attn_mixed_noalloc (static scratch) on the same inputs."""
    tens = make_tensors(batch, seed=seed)
    kc_ref, vc_ref = oracle.kv_append(batch, tens["k_new"], tens["v_new"], tens["k_cache"],
                                      tens["v_cache"])
    ref = oracle.attn(batch, tens["q"], kc_ref, vc_ref)
    t = {k: v.to("cuda") for k, v in tens.items()}
    d = cp.desc_for(batch)
    ws = torch.empty(cp.workspace_bytes(d, batch.rows), dtype=torch.uint8, device="cuda")
    shape = (batch.num_tokens, batch.num_q_heads, batch.head_dim)
    out_ws = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    out_na = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    cp.kv_append(d, t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["block_tables"],
                 batch.rows, ws)
    cp.attn_mixed(d, t["q"], t["k_cache"], t["v_cache"], t["block_tables"], batch.rows, out_ws, ws)
    lib = binding.load()
    r = np.ascontiguousarray(batch.rows)
    rc = lib.cp_attn_mixed_noalloc(ctypes.byref(d), t["q"].data_ptr(), t["k_cache"].data_ptr(),
                                   t["v_cache"].data_ptr(), t["block_tables"].data_ptr(),
                                   r.ctypes.data, r.shape[0], out_na.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
    assert rc == binding.CP_OK, binding.strerror(rc)
    torch.cuda.synchronize()
    return out_ws, out_na, ref


@pytest.mark.gpu
def test_noalloc_matches_attn_mixed_on_two_calls():
    print("[gpu] noalloc: init", flush=True)
    lib = binding.load()
    assert lib.cp_noalloc_init() == binding.CP_OK
    assert lib.cp_noalloc_init() == binding.CP_OK          # idempotent
    # first a full-size mix (27 MB of workspace: split prefill and decode
    # partials), then a smaller batch over the same scratch
    for what, batch, seed in (("mix 2", make_config(2), 8801),
                              ("small", make_batch("small", 8, 2, 64, 32,
                                                   [(300, 70), (0, 1), (129, 1), (5, 9)],
                                                   np.random.default_rng(3)), 8802)):
        d = cp.desc_for(batch)
        print(f"[gpu] noalloc: {what} T={batch.num_tokens} "
              f"ws={cp.workspace_bytes(d, batch.rows)}", flush=True)
        out_ws, out_na, ref = _run_both(batch, seed)
        assert torch.equal(out_ws.view(torch.int16), out_na.view(torch.int16)), \
            f"{what}: noalloc output differs from cp_attn_mixed"
        g = out_na.float().cpu().numpy().astype(np.float64)
        e = np.abs(g - ref)
        print(f"[gpu] noalloc {what}: max_abs={e.max():.3e} mean_abs={e.mean():.3e}", flush=True)
        assert np.isfinite(g).all() and e.max() <= MAX_ABS and e.mean() <= MEAN_ABS


@pytest.mark.gpu
def test_noalloc_with_the_plan_that_fits():
    """The other plan's output.  Each is within 2.3e-3 (2-norm) of the exact one
    (bf16 weights and output), so that they differ by at most about 5e-3."""
    assert binding.load().cp_noalloc_init() == binding.CP_OK
    batch = _two_plans_batch()
    print(f"[gpu] noalloc two plans T={batch.num_tokens}", flush=True)
    t = {k: v.to("cuda") for k, v in make_tensors(batch, seed=8803).items()}
    d = cp.desc_for(batch)
    need = cp.workspace_bytes(d, batch.rows)
    assert need > binding.NOALLOC_SCRATCH_BYTES
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out_ws = torch.empty(batch.num_tokens, 64, 128, dtype=torch.bfloat16, device="cuda")
    out_na = torch.full_like(out_ws, float("nan"))
    cp.kv_append(d, t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["block_tables"],
                 batch.rows, ws)
    cp.attn_mixed(d, t["q"], t["k_cache"], t["v_cache"], t["block_tables"], batch.rows, out_ws, ws)
    r = np.ascontiguousarray(batch.rows)
    rc = binding.load().cp_attn_mixed_noalloc(
        ctypes.byref(d), t["q"].data_ptr(), t["k_cache"].data_ptr(), t["v_cache"].data_ptr(),
        t["block_tables"].data_ptr(), r.ctypes.data, r.shape[0], out_na.data_ptr(),
        torch.cuda.current_stream().cuda_stream)
    assert rc == binding.CP_OK, binding.strerror(rc)
    torch.cuda.synchronize()
    diff = (out_na.double() - out_ws.double()).norm() / out_ws.double().norm()
    assert float(diff) <= 5e-3

"""The session kernel (append and observation of short sessions in one
launch), through the C ABI on the device: parity with the oracle, step by
step, over the sizes where it can go wrong (empty, one-token and page-edge
sessions, tile and chunk edges, the largest session its LDS holds), for every
layout, tier and window, and its void steps and append errors.
"""
import sys

import numpy as np
import pytest
import torch

from paper_2607_10582_amd import binding as B
from synth import configs as C

from harness import Pair

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load_library()


def run(p: Pair, steps: int, label: str):
    """Steps against the oracle; every observation one launch that appends
    too (only steps without an observation launch the append kernel)."""
    p.md.profile(("attend", "append", "logits", "mass"))
    for _ in range(steps):
        st = p.step()
    n = {k: p.md.profile_read(k)[1] for k in ("attend", "append", "logits", "mass")}
    assert n["attend"] > 0 and n["append"] == steps - n["attend"] and n["logits"] == 0 and n["mass"] == 0, n
    status = p.device_status()
    assert status == 0, f"device status {status:#x}"
    assert p.free_pages_consistent()
    print(f"[{label}] ok: {st.steps} steps, {st.tokens} token-steps, max rel {st.max_rel}, evicted {st.evicted_pages}, "
          f"launches {n}", flush=True)
    p.close()
    return st


@pytest.mark.parametrize("Hq,Hkv,L", [(1, 1, 1), (4, 1, 3), (12, 2, 1), (12, 2, 5), (16, 2, 4), (15, 1, 2), (16, 1, 2), (32, 8, 2)])
def test_heads_and_rows(Hq, Hkv, L):
    w = C.with_overrides(C.get("small"), L=L, Hq=Hq, Hkv=Hkv, steps=10)
    run(Pair(w, fused=None, planted=24, planted_strength=2.5, query_gain=0.7), 10, f"heads {Hq}/{Hkv} L{L}")


@pytest.mark.parametrize("P", [16, 64])
@pytest.mark.parametrize("aligned", [False, True])
def test_session_sizes(P, aligned):
    # empty, single, tile and page edges, the eight waves' tiles (128 tokens),
    # one chunk a wave (512), and beyond; budgets below, at and above
    n0s = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512, 513]
    w = C.with_overrides(C.get("small"), L=3, Hq=8, Hkv=2, S=len(n0s), n0=None, n0_range=(1, 2), P=P, steps=40,
                         region_aligned=aligned, append_run=3, system_len=20)
    budgets = [0, 0, 5, 16, 10, 63, 30, 65, 64, 100, 129, 300, 400, 513]
    run(Pair(w, n0s=n0s, budgets=budgets, fused=None, check_free_list=True), 40, f"sizes P{P} aligned{int(aligned)}")


@pytest.mark.parametrize("one_call", [False, True])
def test_large_sessions(one_call):
    # several chunks a wave: a batch of 2,900 and 2,100 tokens beside a short
    # session (alone, sessions as long take the other paths)
    n0s = [2900] * 30 + [2100, 70]
    w = C.with_overrides(C.get("small"), L=4, Hq=8, Hkv=2, S=32, n0=None, n0_range=(1, 2), steps=5, system_len=100)
    run(Pair(w, n0s=n0s, budgets=[2700] * 30 + [2000, 70], fused=None, select_compact=one_call,
             oracle_sessions=[0, 17, 30, 31]), 5, "large")


@pytest.mark.parametrize("aligned", [False, True])
@pytest.mark.parametrize("quant", [0.0, 0.3])
def test_window(aligned, quant):
    w = C.with_overrides(C.get("small_aligned" if aligned else "small"), L=2, window=2, obs_interval=2, steps=16,
                         quant_threshold=quant, n0=700)
    run(Pair(w, fused=None, planted=24, planted_strength=2.5, query_gain=0.7), 16, f"window aligned{int(aligned)}")


@pytest.mark.parametrize("P,aligned", [(16, False), (64, False), (16, True)])
def test_quantised_tier(P, aligned):
    w = C.with_overrides(C.get("small_aligned" if aligned else "small"), L=2, Hq=16, Hkv=2, P=P, n0=900,
                         budget_frac=0.6, steps=24, quant_threshold=0.35)
    run(Pair(w, fused=None, planted=24, planted_strength=2.5, query_gain=0.7), 24, f"quant P{P}")


def test_offload_tier():
    from test_gpu_parity import run_offload
    w = C.with_overrides(C.get("small"), L=2, S=3, n0=None, n0_range=(1, 2), steps=40, system_len=60)
    p = Pair(w, n0s=[450, 700, 300], budgets=[225, 300, 200], planted=24, planted_strength=2.5, query_gain=0.7,
             fused=None, offload_pages=8, drop_threshold=1e-3)
    assert p.md.observe_path()["first"] == p.md.observe_path()["steady"] == "session"
    st = run_offload(p, 40, "session-offload")
    assert st.offloaded > 20 and st.recalled > 10


def test_nonfinite_query_voids_the_session():
    w = C.with_overrides(C.get("small"), L=6, S=3, n0=None, n0_range=(1, 2), steps=4)
    p = Pair(w, n0s=[450, 300, 64], budgets=[225, 150, 64], oracle_sessions=[], fused=None)
    c = p.cache
    imp0 = c.importance.clone()
    q, nk, reg, *_ = p.inputs(1)
    q[1, 0, 4, 3, 17] = float("inf")      # [S][W][L][Hq][d]
    p.md.observe(1, q, nk, reg)
    p.md.score()
    p.md.select_compact()
    torch.cuda.synchronize()
    assert p.md.device_status() == B.MD_DEV_NONFINITE
    cnt = p.md.evict_count.cpu().tolist()
    assert cnt[0] > 0 and cnt[1] == 0
    assert c.n_tokens.cpu().tolist()[1] == 301          # the append stands
    ids = c.page_table[1, :19].long()
    assert torch.equal(c.importance[ids], imp0[ids])    # and changes nothing else
    q, nk, reg, *_ = p.inputs(2)
    p.md.observe(2, q, nk, reg)
    p.md.score()
    p.md.select_compact()
    torch.cuda.synchronize()
    assert p.md.device_status() == 0 and p.md.evict_count.cpu().tolist()[1] > 0
    p.close()


def test_observation_without_append_and_empty_free_list():
    w = C.with_overrides(C.get("small"), L=2, S=2, n0=None, n0_range=(1, 2), steps=4)
    p = Pair(w, n0s=[64, 40], budgets=[1000, 1000], oracle_sessions=[], fused=None)
    c = p.cache
    q, nk, reg, *_ = p.inputs(1)
    abar = torch.zeros_like(c.importance)
    p.md.observe(1, q, abar_out=abar)
    torch.cuda.synchronize()
    assert c.n_tokens.cpu().tolist() == [64, 40] and p.md.device_status() == 0
    assert abs(float(abar.sum()) - 2.0) < 1e-4
    c.set_free_pages([])
    p.md.observe(2, q, nk, reg, abar_out=abar)   # session 0's last page is full: no page for its token
    torch.cuda.synchronize()
    assert p.md.device_status() == B.MD_DEV_CAPACITY
    assert c.n_tokens.cpu().tolist() == [64, 41] and int(c.free_count[0]) == 0
    assert abs(float(abar[c.page_table[1, :3].long()].sum()) - 1.0) < 1e-4
    p.close()


@pytest.mark.parametrize("n,quant,aligned", [(64, 0.0, False), (600, 0.0, False), (640, 0.0, True), (640, 10.0, False)])
def test_window_with_very_low_logits(n, quant, aligned):
    # Every logit of two (layer, KV head) near -150 (a shift of their softmax
    # rows): a chunk whose tokens an older query does not see (the appended
    # token alone in it, for n a multiple of 64) weighs nothing in its row.
    from test_gpu_tail_groups import LOW, run as two_steps
    kw = dict(window=2, quant=quant, aligned=aligned, low=True)
    a, _ = two_steps([n, 200], 2, 8, 2, 16, True, fused=None, **kw)
    b, _ = two_steps([n, 200], 2, 8, 2, 16, True, fused=False, **kw)
    for x, y in zip(a, b):
        for u, v in zip(x[:3], y[:3]):
            assert not np.isnan(u).any() and not np.isnan(v).any()
            fin = np.isfinite(v)
            assert np.array_equal(np.isfinite(u), fin)
            np.testing.assert_allclose(u[fin], v[fin], rtol=LOW, atol=1e-30)


@pytest.mark.parametrize("S,aligned", [(600, False), (1024, True)])
def test_more_sessions_than_threads_and_cus(S, aligned):
    # the commit takes two sessions per thread beyond 512, and the
    # workgroups (one per session) run in several rounds over the CUs
    n0s = [17 + (7 * s) % 48 for s in range(S)]
    w = C.with_overrides(C.get("small"), S=S, n0=None, n0_range=(1, 2), Hq=4, Hkv=1, steps=4, system_len=8,
                         region_aligned=aligned, append_run=3)
    p = Pair(w, n0s=n0s, budgets=[n - 1 - s % 9 for s, n in enumerate(n0s)], fused=None,
             oracle_sessions=[0, 1, 299, 511, 512, 513, S - 2, S - 1], check_free_list=True)
    run(p, 4, f"{S} sessions")


def test_two_handles_of_different_capacity_step_in_turn():
    # one instantiation, two sizes of its LDS: the smaller handle comes
    # second, and neither depends on the order
    w = C.with_overrides(C.get("small"), L=4, steps=4)
    a = Pair(C.with_overrides(w, n0=900), fused=None, max_pages=256)   # room for 4,096 tokens
    b = Pair(C.with_overrides(w, n0=300), fused=None)
    for p in (a, b):
        p.md.profile(("attend", "append"))
    for _ in range(4):
        a.step()
        b.step()
    for p in (a, b):
        assert p.md.profile_read("attend")[1] == 4 and p.md.profile_read("append")[1] == 0
        assert p.device_status() == 0
        p.close()



@pytest.mark.parametrize("S,n0,window,steady", [
    (1, 1500, 1, "session"), (2, 2800, 1, "fused"), (12, 1600, 1, "session"), (96, 105, 1, "fused"),
    (96, 105, 2, "fused"), (4, 500, 2, "session")])
def test_the_session_kernel_is_picked_where_it_is_the_faster_one(S, n0, window, steady):
    # 72 rows (3B shape; half the heads under a window): not for a few long
    # sessions, whose ends one CU adds up, nor for many of a few tokens, each
    # of whose rows has its fixed cost
    w = C.with_overrides(C.get("small"), L=36, Hq=16 // window, Hkv=2, S=S, n0=None, n0_range=(1, 2), window=window,
                         obs_interval=window, steps=2, system_len=8)
    p = Pair(w, n0s=[n0] * S, budgets=[n0 - 1] * S, oracle_sessions=[0], fused=None, max_pages=200)
    assert p.md.observe_path()["steady"] == steady
    for _ in range(2):
        p.step()
    assert p.device_status() == 0
    p.close()


def test_a_session_that_outgrows_the_kernel_leaves_it():
    # one session of two rows is left to the multi-kernel path from about
    # 1,600 tokens on: steps on either side of the change, and a step without
    # an observation between them, match the oracle
    w = C.with_overrides(C.get("small"), n0=1540, steps=90, obs_interval=2)
    p = Pair(w, budgets=[4000], fused=None, max_pages=256)
    assert p.md.observe_path()["steady"] == "session"
    at = None
    for k in range(90):
        p.step()
        if at is None and p.md.observe_path()["steady"] != "session":
            at = k
    assert at is not None and 10 < at < 80
    assert p.md.observe_path()["steady"] == "multi-kernel"
    p.md.profile(("attend", "logits"))
    p.step()
    p.step()
    assert p.md.profile_read("attend")[1] == 0 and p.md.profile_read("logits")[1] == 1
    assert p.device_status() == 0 and p.free_pages_consistent()
    p.close()


@pytest.mark.parametrize("max_pages,steady", [(64, "session"), (256, "multi-kernel")])
def test_an_empty_session_counts_as_full(max_pages, steady):
    w = C.with_overrides(C.get("small"), n0=0, steps=40)
    p = Pair(w, n0s=[0], budgets=[4000], fused=None, max_pages=max_pages)
    assert p.md.observe_path()["steady"] == steady
    for _ in range(40):
        p.step()
    assert p.device_status() == 0
    p.close()


def test_prompts_that_are_never_compacted_keep_their_path():
    # one prompt of 2,600 tokens (56 rows) is too long for the session kernel,
    # what its budget leaves of it is not: observed and selected again and
    # again it stays on the other path, until a selection is applied
    w = C.with_overrides(C.get("small"), L=28, S=1, n0=None, n0_range=(1, 2), steps=6)
    p = Pair(w, n0s=[2600], budgets=[600], oracle_sessions=[], fused=None)
    path = p.md.observe_path()
    assert path["first"] != "session" and path["steady"] == "session"
    p.md.profile(("append",))
    for k in range(1, 6):
        q, nk, reg, *_ = p.inputs(k)
        p.md.observe(k, q, nk, reg)
        p.md.score()
        p.md.select()
        assert p.md.profile_read("append")[1] == (1 if k < 5 else 0), k
        if k == 4:
            p.md.compact()
    assert p.md.device_status() == 0
    p.close()

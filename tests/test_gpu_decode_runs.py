"""Decode attention cut into runs of equal length over requests and kv heads: run lengths from the shortest to several
requests per run, requests cut into many runs, more requests than one scan places, and the batch whose outputs are not
merged, with contexts on both sides of the 32-key pairs and of the 1024 keys whose page ids are read at once: sampled
requests of each batch against the oracle, at the parity bar of the other cases."""
import numpy as np
import pytest
import torch

from paper_2507_06608_amd import synth

from tests.parity_util import assert_close, f32, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nx():
    from paper_2507_06608_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def oracle():
    import oracle
    oracle.lib()
    return oracle


# (requests, contexts that are always there, largest other context): 8 kv heads each
CASES = [
    ("whole contexts, no merge", 5, [0, 15, 16, 254, 255], 255),
    ("shortest runs", 3, [63, 64, 65], 700),
    ("one long request", 1, [8191], 8191),
    ("runs of two pairs", 16, [31, 32, 33, 127, 128, 129], 1000),
    ("runs longer than a window of page ids", 24, [1022, 1023, 1024, 1055, 1056, 8190], 8191),
    ("several requests a run", 300, [0, 31, 32, 1023, 1024, 2047, 2048], 2060),
    ("more requests than one scan", 600, [1022, 1023, 1024, 1025, 0], 1100),
]


@pytest.mark.parametrize("name,n,edges,top", CASES, ids=[c[0] for c in CASES])
def test_equal_runs(nx, oracle, name, n, edges, top):
    print(f"[case] decode attention, {name}", flush=True)
    sh = synth.SHAPES["tiny"]
    rng = np.random.default_rng(n)
    ctx_lens = edges + rng.integers(0, top + 1, n - len(edges)).tolist()
    wl = synth.make_workload(name, sh, 5, chunk_lens=[], prefix_lens=[], decode_ctx=ctx_lens, kv_device="cuda:0")
    w = synth.make_weights(sh, 5)
    ctx = nx.context_for(wl)
    ctx.load_layer(0, w)
    kv = ctx.make_kv(wl.k_pool, wl.v_pool)
    db = nx.DevDecode(wl.decode, ctx.device)
    torch.cuda.synchronize()
    ctx.decode_step(db, kv)
    ctx.sync()
    sampled = sorted(set(range(len(edges))) | {n // 2, n - 1})
    sub = synth.subset_for_oracle(wl, [], sampled)
    ref = run_oracle(oracle, sub, w)
    assert_close(name, f32(db.y[sampled]), ref["y_d"])
    assert torch.isfinite(db.y.float()).all()
    ctx.close()

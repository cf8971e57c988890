"""Every tile shape of the tiled GEMM against every other, bit for bit: per element they add the same products in the same
order, so any shape must reproduce a chunk's outputs exactly, with ragged token counts (partial token tiles), widths that
are no multiple of the tile (partial feature tiles), one to four K slices, every epilogue (a down projection in one slice
adds the residual itself) and K ranges from two stages of the ring up, shorter than the ring that they are loaded into.
The small shapes' default runs are checked against the oracle at the parity bar of the other cases."""
import pytest
import torch

from paper_2507_06608_amd import synth

from tests.parity_util import assert_close, f32, run_oracle
from tests.test_gpu_parity import EXTRA_SHAPES

pytestmark = pytest.mark.gpu

# K = 64 (two stages of 32) in the QKV and gate/up projections, 128 in the other two
SMALL = dict(EXTRA_SHAPES, tiny=synth.SHAPES["tiny"], k64=synth.ModelShape("k64", 64, 2, 2, 64, 96, 10000.0))
TILES = ["128", "128d", "192x128", "256x128", "320x128", "192x256", "256", "320"]


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


@pytest.mark.parametrize("shape,chunks", [("tiny", [129]), ("tiny", [200, 133]), ("llama3_8b", [131]), ("qwen25_14b", [300, 77]), ("llama3_8b", [1033]),
                                          ("gqa5", [190, 71]), ("gqa8", [300]), ("k64", [150, 61])],
                         ids=["tiny 129", "tiny 333", "8B 131", "14B 377", "8B 1033", "one down slice, K 736", "one down slice, K 512", "K 64"])
def test_all_tile_shapes_agree(nx, oracle, monkeypatch, shape, chunks):
    sh = SMALL[shape] if shape in SMALL else synth.SHAPES[shape]
    wl = synth.make_workload("tiles", sh, 3, chunk_lens=chunks, prefix_lens=[17] * len(chunks), decode_ctx=[], kv_device="cuda:0")
    w = synth.make_weights(sh, 3)

    def run(tiles):
        print(f"[case] {shape} {chunks} tiles {tiles}", flush=True)
        if tiles:
            monkeypatch.setenv("NEXUS_GEMM_TILES", tiles)
        else:
            monkeypatch.delenv("NEXUS_GEMM_TILES", raising=False)
        ctx = nx.context_for(wl)
        ctx.load_layer(0, w)
        kv = ctx.make_kv(wl.k_pool, wl.v_pool)
        pb = nx.DevPrefill(wl.prefill, ctx.device)
        torch.cuda.synchronize()
        ctx.prefill_chunk(pb, kv)
        ctx.sync()
        y = pb.y.clone()
        ctx.close()
        return y

    y = run(None)
    if shape in SMALL:
        ref = run_oracle(oracle, wl, w)
        assert_close(f"{shape} {chunks}", f32(y), ref["y_p"])
    for tiles in TILES:
        assert torch.equal(run(tiles).view(torch.int16), y.view(torch.int16)), tiles


def test_an_unknown_tile_shape_is_refused(nx, monkeypatch):
    """A name that is no shape would silently compare the default with itself."""
    print("[case] unknown tile shape", flush=True)
    monkeypatch.setenv("NEXUS_GEMM_TILES", "128x129")
    with pytest.raises(nx.NexusError, match="128x129"):
        nx.Nexus(synth.SHAPES["tiny"], max_prefill_tokens=256, max_prefill_reqs=1, max_decode_reqs=1, max_positions=256)


# Tiles and blocks of tokens of the projections.  Two blocks of tokens that fit 192 CUs, slices and all, are dealt in ranges there; the
# others run in launch order everywhere.
@pytest.mark.parametrize("shape,chunks,tiles", [("tiny", [200, 133], "256"), ("tiny", [257], "320"), ("llama3_8b", [512], "320"), ("qwen25_14b", [257], "320"),
                                                ("qwen25_14b", [129], "320x128"), ("tiny", [129], "256"), ("tiny", [200, 133], "192x128"), ("qwen25_14b", [300, 77], "192x128"),
                                                ("qwen25_14b", [700], "256"), ("llama3_8b", [700], "320x128")],
                         ids=["12, 4 and 22 tiles of two blocks", "10, 4 and 18 of two", "180 of two", "174 of two", "174 of two, 128 tokens", "6, 2 and 11 of one block",
                              "24, 9 and 45 of three", "three blocks", "84, 60 and 324 of three", "six blocks, three slices"])
def test_grids_that_are_no_multiple_of_the_xcds(nx, monkeypatch, shape, chunks, tiles):
    """In either order every tile is computed, with the same bits on the whole chip and on shares.  Another chunk runs through the
    context before each run, so that what a left-out tile would leave behind is wrong (the workspace keeps every intermediate)."""
    print(f"[case] ragged grid {shape} {chunks} {tiles}", flush=True)
    monkeypatch.setenv("NEXUS_GEMM_TILES", tiles)
    sh = synth.SHAPES[shape]
    wl, other = (synth.make_workload("ragged", sh, seed, chunk_lens=chunks, prefix_lens=[9] * len(chunks), decode_ctx=[], kv_device="cuda:0") for seed in (5, 6))
    ctx = nx.context_for(wl)
    ctx.load_layer(0, synth.make_weights(sh, 5))
    kv, kv_other = ctx.make_kv(wl.k_pool, wl.v_pool), ctx.make_kv(other.k_pool, other.v_pool)
    pb, pb_other = nx.DevPrefill(wl.prefill, ctx.device), nx.DevPrefill(other.prefill, ctx.device)

    def run(split, batch, pools):
        ctx.set_cu_split(*split)
        batch.y.fill_(float("nan"))
        torch.cuda.synchronize()
        ctx.prefill_chunk(batch, pools)
        ctx.sync()
        return batch.y.clone()

    whole = (nx.CUS_ALL, nx.CUS_ALL)
    out = []
    for split in (whole, (192, 64), (96, 160)):
        before = run(whole, pb_other, kv_other)
        out.append(run(split, pb, kv))
        assert not torch.isclose(before.float(), out[-1].float()).all(dim=1).any(), "the other chunk has to leave other values"
    ctx.close()
    assert torch.isfinite(out[0].float()).all()
    for y in out[1:]:
        assert torch.equal(y.view(torch.int16), out[0].view(torch.int16))

"""The sizes at which a call changes its plan or kernel, against the oracle (bars as in gpuutil)."""
import pytest
import torch

import test_gpu_parity as parity
from paper_2606_13097_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    yield


@pytest.mark.parametrize("n_seqs,n_segs,page,alias", [(1, 32, 0, False), (1, 33, 0, False), (1, 32, 16, True),
                                                      (65, 1, 16, True), (130, 1, 16, False)])
def test_graft_plan_by_value_and_uploaded(n_seqs, n_segs, page, alias):
    """Up to 32 segments of a graft go by value, more through the staging ring; page rows of up to
    64 sequences go up in one launch, more in several."""
    lengths = [1 + (37 * i) % 131 for i in range(max(n_segs, 5))]
    segs = [[(s + j) % len(lengths) for j in range(n_segs)] for s in range(n_seqs)]
    w = synth.custom(synth.Shape(2, 8, 2, 64, 1e4, "bf16"), 3, lengths, segs, 5, 1, page_size=page)
    parity.run_pipeline(w, [1], 1, [0, n_seqs - 1], alias=alias)


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("last", [2048, 2049])
def test_graft_of_as_many_runs_as_go_by_value(last, page):
    """32 segments in 1024 runs of 64 tokens go by value, one token more through the staging ring."""
    segs = [[0, 1, 2, 3]] * 7 + [[0, 1, 2, 4]]
    w = synth.custom(synth.Shape(1, 2, 1, 64, 1e4, "bf16"), 4, [2048] * 4 + [last], segs, 1, 1, page_size=page)
    parity.run_pipeline(w, [0], 1, [0, 7])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g,page,alias", [(1, 0, False), (2, 16, True), (4, 16, False), (8, 0, False), (16, 16, True)])
@pytest.mark.parametrize("ctx", ["edges", "long"])
def test_decode_ring_and_merge(d, g, page, alias, ctx):
    """Both rings of the bf16 decode (one short split per CU; two blocks per CU past 256 keys for
    each) at ragged lengths: fewer tiles than waves, a partial tile, a split that holds the new
    token alone, a sequence of many splits."""
    if ctx == "edges":
        hkv, lens = 2, [1, 15, 63, 64, 127, 800, 191]
    else:
        hkv, lens = (8, [8301, 17, 1535]) if g < 16 else (4, [16601, 17, 1535])  # over 65536 (key, kv head) pairs
    # two fresh tokens precede the decode steps: segment lengths two short
    segs = [[i] for i in range(len(lens))]
    w = synth.custom(synth.Shape(1, hkv * g, hkv, d, 1e6, "bf16"), 5, [max(1, n - 2) for n in lens], segs, 2, 3,
                     page_size=page)
    parity.run_pipeline(w, [0], 3, list(range(len(lens))), alias=alias)


@pytest.mark.parametrize("g,d,ctx", [(4, 128, 2990), (2, 64, 9990), (8, 64, 4100), (16, 64, 2100)])
@pytest.mark.parametrize("page", [0, 16])
def test_decode_merge_in_several_batches(g, d, ctx, page):
    """One kv head, so splits of 64 keys: more of them (47, 157, 65, 33) than the merge's lanes fetch
    at a time (8 per lane: 32, 128, 32, 16), as many lanes to a chunk as the instance has (4, 16, 4, 2)."""
    w = synth.custom(synth.Shape(1, g, 1, d, 1e6, "bf16"), 15, [ctx], [[0]], 1, 2, page_size=page)
    parity.run_pipeline(w, [0], 2, [0])


@pytest.mark.parametrize("g,d,page,alias", [(4, 128, 0, False), (16, 64, 16, True), (1, 128, 16, False)])
def test_decode_of_many_short_sequences(g, d, page, alias):
    """Few keys but more blocks than CUs, most of them empty (one long sequence): the ring of two."""
    lens = [5, 33, 61, 900] + [9] * 36
    w = synth.custom(synth.Shape(1, 2 * g, 2, d, 1e6, "bf16"), 16, lens, [[i] for i in range(len(lens))], 2, 2,
                     page_size=page)
    parity.run_pipeline(w, [0], 2, [0, 1, 2, 3, 39], alias=alias)


@pytest.mark.parametrize("g,d", [(1, 64), (2, 128), (8, 64), (16, 128)])
def test_fp32_decode_merge(g, d):
    """The fp32 step's split merge over its chunk counts (16 to 512 16-byte chunks a split), with a
    sequence of one split and one of many."""
    w = synth.custom(synth.Shape(1, 2 * g, 2, d, 1e4, "f32"), 5, [40, 3000], [[0], [1]], 2, 2, page_size=0)
    parity.run_pipeline(w, [0], 2, [0, 1])


@pytest.mark.parametrize("d,g", [(64, 2), (128, 4), (128, 16)])
@pytest.mark.parametrize("page,alias", [(0, False), (16, False), (16, True)])
@pytest.mark.parametrize("n_fresh", [1, 40, 131])
def test_prefill_tile_addresses(d, g, page, alias, n_fresh):
    """Key tiles wholly cached (addressed from a scalar base per load) and tiles that hold fresh
    keys or end the split (per lane), with contexts around multiples of the 64-key tile."""
    lens = [1, 63, 64, 65, 127, 449]
    w = synth.custom(synth.Shape(1, 2 * g, 2, d, 1e6, "bf16"), 7, lens, [[i] for i in range(len(lens))], n_fresh, 1,
                     page_size=page)
    parity.run_pipeline(w, [0], 1, list(range(len(lens))), alias=alias)


@pytest.mark.parametrize("d,g", [(64, 1), (64, 2), (64, 4), (64, 8), (64, 16), (128, 1), (128, 2), (128, 4),
                                 (128, 8), (128, 16)])
@pytest.mark.parametrize("page,alias", [(0, False), (16, True)])
@pytest.mark.parametrize("n_fresh,lens", [(1, [1, 127, 128, 700]), (7, [1, 57, 63, 121, 122, 700]),
                                          (131, [1, 900, 2500, 2600])])
def test_fp32_prefill_row_blocks(d, g, page, alias, n_fresh, lens):
    """The fp32 prefill over 1, 2 and 4 tokens a block (few and many blocks a call), blocks of fewer
    tokens than that, key splits of one and of several tiles, contexts around multiples of a step."""
    w = synth.custom(synth.Shape(1, 2 * g, 2, d, 1e4, "f32"), 9, lens, [[i] for i in range(len(lens))], n_fresh, 1,
                     page_size=page)
    parity.run_pipeline(w, [0], 1, list(range(len(lens))), alias=alias)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_kept", [2, 40])
def test_graft_aliases_a_page_a_cut_left_mapped(dtype, n_kept, monkeypatch):
    """A segment grafted behind a gap and cut away again leaves the cut page mapped and empty; a
    segment that then covers the page reads its values from the library though the call maps no new
    page of that sequence (up to 32 segments, by value, and more, uploaded)."""
    from paper_2606_13097_amd import fcg, runner
    plain = runner.GpuSetup.graft

    def graft(self):
        for s in range(n_kept):
            fcg.fcg_graft(self.cache, self.lib, [s], [0], [5])
            fcg.fcg_cache_truncate(self.cache, s, 5)
        plain(self)

    monkeypatch.setattr(runner.GpuSetup, "graft", graft)
    # no fresh tokens: a prefill that maps a page would bring the row up to date
    check = parity.check_attn
    monkeypatch.setattr(parity, "check_attn", lambda got, *a: check(got, *a) if got.size else None)
    w = synth.custom(synth.Shape(2, 4, 2, 64, 1e4, dtype), 11, [8, 16, 37], [[1]] * n_kept + [[2]], 0, 3, page_size=16)
    parity.run_pipeline(w, [1], 3, [0, n_kept - 1, n_kept], alias=True)


@pytest.mark.parametrize("dtype,d,g,page,shift", [("bf16", 128, 4, 0, 1), ("bf16", 128, 4, 0, 4), ("bf16", 64, 1, 16, 1),
                                                  ("bf16", 128, 16, 16, 2), ("f32", 64, 2, 0, 1)])
def test_tensors_at_any_element(dtype, d, g, page, shift, monkeypatch):
    """q, k, v and out that start at any element of a buffer (a multiple of 16 bytes selects the loads
    straight into LDS, others the ordinary ones)."""
    from paper_2606_13097_amd import fcg

    def moved(t):
        buf = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)
        buf[shift:].copy_(t.reshape(-1))
        return buf[shift:].view(t.shape)

    def shifted(fn, n_lead):
        def call(*args):
            q, k, v, out = (moved(t) for t in args[n_lead:])
            assert q.data_ptr() % 16
            res = fn(*args[:n_lead], q, k, v, out)
            args[-1].copy_(out)
            return res
        return call

    monkeypatch.setattr(fcg, "fcg_patch_prefill", shifted(fcg.fcg_patch_prefill, 4))
    plain_decode = shifted(fcg.fcg_decode, 3)
    monkeypatch.setattr(fcg, "fcg_decode", lambda *a: plain_decode(*a[:7]))   # the runner passes a stream, None
    w = synth.custom(synth.Shape(1, 2 * g, 2, d, 1e4, dtype), 13, [70, 800], [[0], [1]], 9, 3, page_size=page)
    parity.run_pipeline(w, [0], 3, [0, 1])

"""Kernel edges on the GPU: tile remainders, split and dispatch boundaries, against the fp64 oracle.

One-layer models of small odd widths, run through prefill and teacher-forced decode.  Bars as in the
other parity tests: bf16 logits within 2e-2 of the oracle per position (a bf16 layer of these widths is
0.3-1% from it), fp32 within 1e-4, ids equal wherever the oracle's top-2 margin exceeds that.
"""
import dataclasses

import numpy as np
import pytest

from oracle import model as om
from tests.gpu_helpers import decode_items, rp, teacher_forced_parity
from workloads import ModelShape, make_weights, weights_to_numpy
from workloads.gen import Workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
SMALL = ModelShape("small", 1, 384, 6, 2, 64, 640, 1152, False, "bf16")


def _workload(shape, plens, seed):
    rng = np.random.default_rng(seed)
    prompts = [rng.integers(0, shape.vocab, size=int(p)).astype(np.int32) for p in plens]
    offs = np.concatenate([[0], np.cumsum([len(p) for p in prompts])]).astype(np.int64)
    n = len(prompts)
    return Workload("edges", shape, np.arange(500, 500 + n, dtype=np.int64), np.concatenate(prompts), offs,
                    np.ones(n, np.int32), np.arange(n, dtype=np.int32), 1.0, 11)


def _parity(shape, plens, n_new, max_prefill, tol=2e-2, check=None, pack=True):
    wd = make_weights(shape, seed=3, device=DEV)
    w64 = weights_to_numpy(wd)
    wl = _workload(shape, plens, len(plens) + sum(plens))
    ctx = max(plens) + n_new
    R = rp()
    eng = R.Engine(shape, R.weights_for_engine(wd), max_seqs=len(plens), max_prefill_tokens=max_prefill,
                   max_context=ctx, kv_pages=sum((p + n_new + 63) // 64 for p in plens), pack_weights=pack)
    r = teacher_forced_parity(eng, shape, w64, wl, n_new, tol, 1.0, 11, check=check)
    eng.close()
    assert r.max_rel_err <= tol and r.id_mismatch == 0, r


@pytest.mark.parametrize("rows", [65, 96, 127, 128, 129, 255, 256, 257, 385, 513])
def test_tiled_gemm_row_edges(rows):
    """Decode batches around the tiled GEMM's 128- and 256-row tiles, prefilled from prompts of 1-3
    tokens, so that most rows of the prefill tiles are some sequence's last and are compared too.
    640 and 1,152 weight rows leave ragged panels, K = 384 and 640 six and ten K steps.  The engine
    of every second case holds one split's partials only, which caps the K splits of the prefill."""
    plens = [1 + i % 3 for i in range(rows)]
    _parity(SMALL, plens, 2, max_prefill=sum(plens) if rows % 2 else 4096)


@pytest.mark.parametrize("hd,inter,vocab,plens", [
    (64, 75, 301, [1, 7, 16]),                       # K = 75: element loads; ragged 16-row tiles
    (128, 76, 320, [64, 65, 129] + [5] * 14),        # 17 rows: two activation tiles; page edges
    (64, 690, 1001, [321, 260, 3] + [2] * 37),       # 40 rows, four tiles; contexts of more pages than waves
    (128, 132, 130, [700]),                          # one row, eleven pages
])
def test_fp32_model_edges(hd, inter, vocab, plens):
    """fp32 products with ragged N, K that is no multiple of 4 or 16, 1 to 64+ activation rows, and
    attention over one to eleven pages (four waves per row share them).  fp32 sums of up to 690
    products of either order agree to about 1e-6; the bar is the fp32 model's 1e-4."""
    shape = ModelShape("f32", 2, 132, 6, 2, hd, inter, vocab, False, "f32")
    _parity(shape, plens, 3, max_prefill=2048, tol=1e-4)


@pytest.mark.parametrize("n_q,n_kv,hd,plens", [
    (14, 2, 64, [1, 31, 32, 33, 62, 63, 64, 65, 126, 127, 128, 129]),  # half-page and page edges, one item a row
    (7, 1, 128, [255, 256, 257, 511, 640, 1]),                         # several half pages a wave
    (16, 1, 64, [64, 40]),                                             # 16 query heads: every column used
    (3, 3, 128, [130, 2]),                                             # one query head per KV head
    (14, 2, 64, [2300] + [5, 64] * 3),                                 # a long row in items beside single ones
    (4, 4, 128, [1500, 1400, 63]),                                     # few rows: items and the 1024-thread merge
    (16, 16, 64, [1, 31, 32, 33, 63, 64, 65, 127, 128, 129] * 13),     # 2,080 short items: one wave each
    (12, 12, 128, [1, 31, 32, 33, 63, 64, 65, 130, 200] * 19),         # 2,052 of them at head dim 128
    (16, 16, 64, [2100] + [40] * 127),                                 # 2,096, one row of four items
])
def test_decode_attention_edges(n_q, n_kv, hd, plens):
    """Decode attention items: cached keys ending on and beside half pages and pages (the newest
    token opens a page), waves without a half page, one to sixteen query heads per KV head, rows of
    one item and of several, which the merge combines."""
    shape = ModelShape("attn", 1, 384, n_q, n_kv, hd, 256, 640, False, "bf16")
    if (n_q + 2 * n_kv) * hd % 128 or n_q * hd % 128:
        shape = dataclasses.replace(shape, n_q=n_q, head_dim=128)
    _parity(shape, plens, 3, max_prefill=4096)


@pytest.mark.parametrize("rows", [1, 8, 9, 16, 17, 31, 32, 33, 48, 49, 63, 64])
@pytest.mark.parametrize("pack", [True, False])
def test_decode_gemm_row_edges(rows, pack):
    """Decode batches around the 16-row activation tiles of the ring GEMM and its 9- and 17-row rules,
    packed and row-major weights.  Six and ten K units leave waves with one, two or three units, 640
    and 1,152 weight rows ragged last blocks."""
    _parity(SMALL, [1 + i % 5 for i in range(rows)], 3, max_prefill=1024, pack=pack)


@pytest.mark.parametrize("rows,pack", [(3, True), (3, False), (16, True), (40, False), (64, True), (397, True)])
def test_decode_gemm_wide(rows, pack):
    """The 7B layer's K = 3,584 and 18,944 (fourteen and dozens of units per wave, K splits, the ring at few
    rows) and a ragged head of 8,320 rows; at 397 rows gate/up in two launches of different tiles."""
    shape = ModelShape("wide", 1, 3584, 28, 4, 128, 18944, 8320, False, "bf16")
    _parity(shape, [1 + i % 3 for i in range(rows)], 2, max_prefill=1024, pack=pack, check=[0, rows // 2, rows - 1])


@pytest.mark.parametrize("plens", [[40, 41, 42], [1] * 20])
def test_silu_of_large_negative_gates(plens):
    """SiLU down to where exp(-z) overflows: at gates of -87.3 to -88.7 its values, -1e-36 to -2e-37, are normal
    bf16 numbers.  Gates of -88.5 to -86 on up values of 1e36 give activations of order one, so a
    product that flushed them to zero would miss the oracle's logits by 0.22 (below -88.72 exp(-z) is infinite
    in fp32, and the result zero).  The attention output is zero and every token's hidden state has the same two large entries, which alone meet the gate and up
    weights: the bf16 rounding of the hidden state (the oracle rounds there too) fixes the gates."""
    s = dataclasses.replace(SMALL, vocab=640)
    wd = make_weights(s, seed=5, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(1)
    e = (torch.randint(0, 2, (s.vocab, s.hidden), generator=gen, device=DEV) * 2 - 1) / 64.0
    e[:, 0], e[:, 1] = 1.0, 0.125
    wd["embed"].copy_(e)
    L = wd["layers"][0]
    L["wo"].zero_()
    for k in ("w_gate", "w_up"):
        L[k].zero_()
    h0 = float((1.0 / torch.sqrt((e[0].double() ** 2).mean() + 1e-6)))
    assert abs(h0 / 0.125 % 1.0 - 0.5) > 0.01  # not beside a rounding boundary of bf16 (steps of 1/8 from 16 to 32)
    h0 = round(h0 * 8) / 8
    L["w_gate"][:, 0] = -88.0 / h0
    L["w_gate"][:, 1] = torch.linspace(-0.5, 2.0, s.inter, device=DEV) / (h0 / 8)
    L["w_up"][:, 0] = 1e36 / h0
    gates = L["w_gate"][:, :2].double() @ torch.tensor([h0, h0 / 8], dtype=torch.float64, device=DEV)
    assert float(gates.min()) > -88.6 and int((gates < -87.4).sum()) > 100
    w64 = weights_to_numpy(wd)
    wl = _workload(s, plens, sum(plens))
    R = rp()
    eng = R.Engine(s, R.weights_for_engine(wd), max_seqs=len(plens), max_prefill_tokens=256, max_context=64,
                   kv_pages=len(plens))
    r = teacher_forced_parity(eng, s, w64, wl, 3, 2e-2, 1.0, 11, rnd=om.bf16_round)
    eng.close()
    assert r.max_rel_err <= 2e-2 and r.id_mismatch == 0, r


def test_tiled_gemm_of_more_than_two_million_columns():
    """A head of 4,194,688 rows: 256 rows of fp32 logits span more than 4 GiB, past what a 32-bit offset over
    a whole 256-row tile reaches.  The tiled GEMM's logits (256 prompts at once) against the ring GEMM's, which
    addresses row by row (64 at a time).  The two sum the layer's products in other orders; both are held to 2e-2
    of the oracle elsewhere, so to 4e-2 of each other here."""
    s = ModelShape("wide-head", 1, 128, 2, 2, 64, 128, (1 << 22) + 384, True, "bf16")
    wd = make_weights(s, seed=7, device=DEV)
    R = rp()
    n = 256
    toks = np.random.default_rng(3).integers(0, s.vocab, size=n).astype(np.int32)
    eng = R.Engine(s, R.weights_for_engine(wd), max_seqs=n, max_prefill_tokens=n, max_context=4, kv_pages=n)

    def logits(lo, hi):
        ids = np.arange(lo, hi, dtype=np.int64)
        out, _ = eng.prefill(ids, toks[lo:hi], np.arange(hi - lo + 1, dtype=np.int64), np.full(hi - lo, 2, np.int32),
                             1, 1.0, logits=True)
        eng.abort(ids)
        return out

    whole = logits(0, n)
    for lo in range(0, n, 64):
        part = logits(lo, lo + 64)
        err = (whole[lo:lo + 64] - part).abs().amax(1) / part.abs().amax(1)
        assert float(err.max()) <= 4e-2, (lo, err)
    eng.close()


def test_decode_attention_profile_counts_its_fused_work():
    """bf16 decode steps launch no rotation or append of their own: the attention class carries their
    bytes, the projection's fp32 partials and the K/V of the cached and the new tokens, beside its output; a merge
    is there only where some row has several items."""
    wd = make_weights(SMALL, seed=3, device=DEV)
    R = rp()
    for plens, merges in (([5, 9, 70], 0), ([3000, 9], 1)):
        wl = _workload(SMALL, plens, 1)
        n = len(plens)
        eng = R.Engine(SMALL, R.weights_for_engine(wd), max_seqs=n, max_prefill_tokens=4096, max_context=max(plens) + 4,
                       kv_pages=sum(p // 64 + 1 for p in plens))
        eng.prefill(wl.seq_ids, wl.prompt_tokens, wl.prompt_offsets, np.full(n, 3, np.int32), 1, 1.0)
        eng.profile(["rope_append", "attn", "attn_merge"], every=1)
        eng.decode_step()
        got = {r["kernel"]: r for r in eng.profile_read()}
        eng.close()
        assert (decode_items(SMALL, np.array(plens) + 1)[1].max() > 1) == bool(merges)
        assert "rope_append" not in got and got.get("attn_merge", {"launches": 0})["launches"] == merges
        kv = 2 * SMALL.n_kv * SMALL.head_dim * 2 * sum(p + 1 for p in plens)
        out = n * SMALL.n_q * SMALL.head_dim * 2
        assert got["attn"]["bytes"] == kv + n * SMALL.qkv_out * 4 + out, got

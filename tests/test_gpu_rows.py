"""The matrix products of prompts and batched decode steps at the edges of their
row tiles and launch shapes, bf16 and 8-bit weights, against the float64 oracle: logits, and every cached key and value of every row.

Tolerances: logits 1e-3 of the largest (fp32-accurate activations).  A cached key
or value that lies next to a rounding boundary may round the other way, one bf16
step, at most 2^-7 of it; a row in which every element did would be 2^-7 off in
two-norm, a row or column a tile missed or took twice is of order one off."""

from __future__ import annotations

import numpy as np
import pytest

from oracle import DecoderOracle, q8_model_f64
from paper_2608_24204_amd import configs, inputs
from tests.helpers import inf_rel

pytestmark = pytest.mark.gpu

# narrow: every product split along K (3 and 9 ranges of 128 among them), vocab and
# QKV rows no multiple of a tile; wide: gate/up and LM head past 192 x 128 rows, the
# LM head's last tile ragged; deep: the down product in K ranges of 1024 on 128 weight rows;
# mid: gate/up and LM head of 128 to 192 x 128 rows, which leave the few-row kernel past 64 rows
CFGS = {
    "narrow": configs.ModelConfig(name="t_rows", key=110, n_layers=2, d_model=384, n_heads=4,
                                  n_kv_heads=2, head_dim=64, ffn_dim=1152, vocab=1003),
    "wide": configs.ModelConfig(name="t_rows_wide", key=111, n_layers=2, d_model=256, n_heads=2,
                                n_kv_heads=1, head_dim=128, ffn_dim=12416, vocab=24601),
    "mid": configs.ModelConfig(name="t_rows_mid", key=113, n_layers=1, d_model=256, n_heads=2,
                               n_kv_heads=1, head_dim=128, ffn_dim=8320, vocab=17001),
    "deep": configs.ModelConfig(name="t_rows_deep", key=112, n_layers=1, d_model=2048, n_heads=4,
                                n_kv_heads=1, head_dim=128, ffn_dim=12288, vocab=1003),
    # no product's K a multiple of 128 (every other kernel than the few-row one), and K of
    # two steps, fewer than the stages of the smallest tile
    "odd": configs.ModelConfig(name="t_rows_odd", key=114, n_layers=2, d_model=320, n_heads=5,
                               n_kv_heads=1, head_dim=64, ffn_dim=448, vocab=1003),
    "step": configs.ModelConfig(name="t_rows_step", key=115, n_layers=2, d_model=64, n_heads=1,
                                n_kv_heads=1, head_dim=64, ffn_dim=64, vocab=251),
}

# Every tile with every epilogue at row and column remainders (test_product_plan.py checks
# that these are what the rules choose for these rows): cols for stored and SwiGLU products,
# resid for the residual ones, ranges for K ranges.
TILE_ROWS = {"cols": [200, 333, 600, 1000], "resid": [333, 600, 1000], "ranges": [100, 333, 777]}
TILE_CFGS = {
    "cols": configs.ModelConfig(name="t_cols", key=116, n_layers=2, d_model=1088, n_heads=85,
                                n_kv_heads=17, head_dim=64, ffn_dim=4160, vocab=1003),
    "resid": configs.ModelConfig(name="t_resid", key=117, n_layers=2, d_model=6208, n_heads=20,
                                 n_kv_heads=4, head_dim=128, ffn_dim=1472, vocab=1003),
    "ranges": configs.ModelConfig(name="t_ranges", key=118, n_layers=2, d_model=4032, n_heads=32,
                                  n_kv_heads=4, head_dim=128, ffn_dim=512, vocab=1003),
}


def setup(name, weights):
    cfg = {**CFGS, **TILE_CFGS}[name].with_(weight_dtype=weights)
    w = inputs.make_weights(cfg, gain_std=0.1)
    return cfg, w, (q8_model_f64(w) if weights == "q8" else inputs.weights_f64(cfg, w))


def check_kv(m, orc, n):
    for l in range(m.cfg.n_layers):
        for got, ref in zip(m.read_kv(l, 0, n), (orc.K[l][:n], orc.V[l][:n])):
            got = inputs.bf16_bits_to_f32(got).astype(np.float64).reshape(n, -1)
            ref = ref.reshape(n, -1)
            err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
            assert err.max() <= 2.0 ** -7, (l, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("weights", ["bf16", "q8"])
@pytest.mark.parametrize("name", [n for n in CFGS if n != "mid"])
def test_short_prompts_match_oracle(cuda_ok, name, weights):
    """Prompts of 1 to 129 rows: both sides of every row tile, and of the most rows
    the kernel takes (64 with 8-bit weights, 128 with bf16)."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg, w, w64 = setup(name, weights)
    sizes = [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129]
    toks = np.random.default_rng(3).integers(0, cfg.vocab, sizes[-1]).astype(np.int32)
    orc = DecoderOracle(cfg, w64, max_seq=sizes[-1])
    ref = orc.full(toks)
    m = WiciModel(cfg, max_seq=sizes[-1])
    try:
        m.load_weights(w)
        for n in sizes:
            m.reset_kv()
            tok, lg = m.prefill(toks[:n], want_logits=True)
            print(f"[rows] {name} {weights} {n} rows: {inf_rel(lg, ref[n - 1]):.2e}", flush=True)
            assert inf_rel(lg, ref[n - 1]) <= 1e-3, n
            assert tok == int(np.argmax(lg)), n
            check_kv(m, orc, n)
    finally:
        m.close()


@pytest.mark.parametrize("weights", ["bf16", "q8"])
@pytest.mark.parametrize("name,sizes", [("narrow", [200, 257, 500, 640, 1023, 1024, 1281]),
                                        ("wide", [130, 200, 257, 400])])
def test_long_prompts_match_oracle(cuda_ok, name, sizes, weights):
    """130 to 1281 rows: the tiled products with ragged rows, whole column tiles (384, 512,
    2304 and 24832 columns), split along K and not."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg, w, w64 = setup(name, weights)
    toks = np.random.default_rng(4).integers(0, cfg.vocab, sizes[-1]).astype(np.int32)
    orc = DecoderOracle(cfg, w64, max_seq=sizes[-1])
    ref = orc.full(toks)
    m = WiciModel(cfg, max_seq=sizes[-1])
    try:
        m.load_weights(w)
        for n in sizes:
            m.reset_kv()
            tok, lg = m.prefill(toks[:n], want_logits=True)
            print(f"[rows] {name} {weights} {n} rows: {inf_rel(lg, ref[n - 1]):.2e}", flush=True)
            assert inf_rel(lg, ref[n - 1]) <= 1e-3, n
            check_kv(m, orc, n)
    finally:
        m.close()


@pytest.mark.parametrize("name", list(TILE_CFGS))
def test_ragged_tiles_match_oracle(cuda_ok, name):
    """Every tile with every epilogue, rows and columns no multiple of it: the second
    layer's keys and values show every row and column of the first one's products."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg, w, w64 = setup(name, "bf16")
    sizes = TILE_ROWS[name]
    toks = np.random.default_rng(8).integers(0, cfg.vocab, sizes[-1]).astype(np.int32)
    orc = DecoderOracle(cfg, w64, max_seq=sizes[-1])
    ref = orc.full(toks)
    m = WiciModel(cfg, max_seq=sizes[-1], prefill_chunk=2048)
    try:
        m.load_weights(w)
        for n in sizes:
            m.reset_kv()
            tok, lg = m.prefill(toks[:n], want_logits=True)
            print(f"[rows] {name} {n} rows: {inf_rel(lg, ref[n - 1]):.2e}", flush=True)
            assert inf_rel(lg, ref[n - 1]) <= 1e-3, n
            check_kv(m, orc, n)
    finally:
        m.close()


@pytest.mark.parametrize("weights", ["bf16", "q8"])
@pytest.mark.parametrize("name,n", [("narrow", 9), ("narrow", 17), ("narrow", 48), ("narrow", 64),
                                    ("narrow", 65), ("narrow", 130), ("wide", 3), ("wide", 49), ("wide", 97),
                                    ("mid", 64), ("mid", 65), ("mid", 128), ("odd", 7),
                                    ("odd", 32), ("odd", 40), ("step", 3), ("step", 33)])
def test_batches_match_oracle(cuda_ok, name, weights, n):
    """Batched steps with given tokens, sequences of different lengths."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg, w, w64 = setup(name, weights)
    rng = np.random.default_rng(n)
    kw = dict(max_seq=40, prefill_chunk=256)
    lead = WiciModel(cfg, **kw)
    ms = [lead]
    try:
        lead.load_weights(w)
        ms += [WiciModel(cfg, share_weights_of=lead, **kw) for _ in range(n - 1)]
        ps = [rng.integers(0, cfg.vocab, 1 + b % 7).astype(np.int32) for b in range(n)]
        fed = rng.integers(0, cfg.vocab, (2, n)).astype(np.int32)
        for m, p in zip(ms, ps):
            m.prefill(p)
        lead.decode_batch(ms, fed[0])
        toks, lg = lead.decode_batch(ms, fed[1], want_logits=True)
        worst = 0.0
        for b in range(n):
            orc = DecoderOracle(cfg, w64, max_seq=40)
            ref = orc.forward(np.concatenate([ps[b], fed[:, b]]))
            worst = max(worst, inf_rel(lg[b], ref))
            assert inf_rel(lg[b], ref) <= 1e-3, b
            assert toks[b] == int(np.argmax(lg[b]))
            check_kv(ms[b], orc, len(ps[b]) + 2)
        print(f"[rows] {name} {weights} batch {n}: {worst:.2e}", flush=True)
    finally:
        for m in ms:
            m.close()


def test_batch_groups_change_between_steps(cuda_ok):
    """Descriptors, given tokens and returned states pass through one pinned buffer
    per lead: groups of changing size, order and lead, tokens given for some
    sequences only, with and without logits, each step's tokens and positions as when
    every sequence decodes alone."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg, w, _ = setup("narrow", "bf16")
    kw = dict(max_seq=40, prefill_chunk=256)
    rng = np.random.default_rng(5)
    groups = [[0, 1, 2, 3, 4], [3, 1], [1, 3, 0], [4, 2, 0, 1], [3, 4], [0, 1, 2, 3, 4], [2, 0]]
    given = [[int(t) if rng.random() < 0.5 else -1 for t in rng.integers(0, cfg.vocab, len(g))]
             for g in groups]
    lead = WiciModel(cfg, **kw)
    ms = [lead]
    try:
        lead.load_weights(w)
        ms += [WiciModel(cfg, share_weights_of=lead, **kw) for _ in range(4)]
        ps = [rng.integers(0, cfg.vocab, 3 + b).astype(np.int32) for b in range(5)]

        def run(step):
            out = []
            for m, p in zip(ms, ps):
                m.reset_kv()
                m.prefill(p)
            for i, (g, t) in enumerate(zip(groups, given)):
                out.append(step(i, [ms[b] for b in g], t))
            return out, [m.position for m in ms]

        def batched(i, models, toks):
            got = WiciModel.decode_batch(models, toks, want_logits=i % 2 == 1)
            return [int(t) for t in (got[0] if i % 2 == 1 else got)]

        alone = run(lambda i, models, toks: [m.decode_step(t)[0] for m, t in zip(models, toks)])
        assert run(batched) == alone
        assert run(batched) == alone   # replayed graphs
    finally:
        for m in ms:
            m.close()


@pytest.mark.parametrize("weights", ["bf16", "q8"])
@pytest.mark.parametrize("name", ["narrow", "deep"])
def test_prompts_have_no_in_launch_sum(cuda_ok, name, weights):
    """No product of a prompt, whatever its rows, adds its K ranges within the launch
    (which needs workgroups dealt to the XCDs in turn): with WICI_FLAG_FAULT_DRILL,
    under which every such sum reports misplaced ranges, prompts succeed and their
    results are those without the flag, while the batched step fails."""
    from paper_2608_24204_amd.binding import WICI_E_HIP, WiciError, WiciModel
    cfg, w, _ = setup(name, weights)
    toks = np.random.default_rng(6).integers(0, cfg.vocab, 129).astype(np.int32)

    def run(drill):
        out = []
        lead = WiciModel(cfg, max_seq=160, fault_drill=drill)
        ms = [lead]
        try:
            lead.load_weights(w)
            for n in (1, 16, 33, 64, 65, 128, 129):
                lead.reset_kv()
                out.append(lead.prefill(toks[:n], want_logits=True))
            ms.append(WiciModel(cfg, max_seq=160, share_weights_of=lead))
            ms[1].prefill(toks[:5])
            if drill:
                with pytest.raises(WiciError) as e:
                    lead.decode_batch(ms)
                assert e.value.status == WICI_E_HIP and "XCD" in str(e.value)
        finally:
            for m in ms:
                m.close()
        return out

    for (t0, l0), (t1, l1) in zip(run(False), run(True)):
        assert t0 == t1 and np.array_equal(l0, l1)


@pytest.mark.parametrize("n", [2, 16, 17, 32])
def test_short_prompts_sum_in_quarters_of_k(cuda_ok, n):
    """Three terms throughout and an fp32 cache: what is left is the error of fp32 sums.  m
    additions in a row, each rounded to u = 2^-24 of a partial sum that grows as a random
    walk, are u sqrt(m / 6) off.  Over a quarter of K = 4096 (m = 3 * 1024 / 32 matrix-core
    steps) that is 4.0 u, 2.4e-7, over all of it 4.8e-7; the norm, the rotation and the
    dropped terms are about as much again as the former: 5.7 u in all, bound 6.7 u, and
    three times that behind the layer's other three products."""
    from paper_2608_24204_amd.binding import WiciModel
    cfg = configs.ModelConfig(name="t_sums", key=119, n_layers=2, d_model=4096, n_heads=32,
                              n_kv_heads=8, head_dim=128, ffn_dim=2048, vocab=1003,
                              kv_dtype="f32")
    w = inputs.make_weights(cfg, gain_std=0.1)
    toks = np.random.default_rng(9).integers(0, cfg.vocab, n).astype(np.int32)
    orc = DecoderOracle(cfg, inputs.weights_f64(cfg, w), max_seq=n)
    orc.full(toks)
    m = WiciModel(cfg, max_seq=n, prefill_mode="bf16x3")
    try:
        m.load_weights(w)
        m.prefill(toks)
        err = []
        for l in range(2):
            got = np.concatenate([z.reshape(n, -1) for z in m.read_kv(l, 0, n)]).astype(np.float64)
            want = np.concatenate([z[:n].reshape(n, -1) for z in (orc.K[l], orc.V[l])])
            err.append(np.linalg.norm(got - want) / np.linalg.norm(want))
        print(f"[rows] sums {n} rows: keys and values {err[0]:.2e} {err[1]:.2e}", flush=True)
        assert err[0] <= 6.7 * 2.0 ** -24 and err[1] <= 20 * 2.0 ** -24
    finally:
        m.close()

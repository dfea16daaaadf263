"""GPU parity at the edges of the launch rules: sizes and options on both sides
of each choice between kernels, against the fp64 oracle."""
import pytest

from paper_2606_07878_amd import configs, synth
from tests.helpers import BF16_TOL, FP32_TOL, assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _layer_case(w, mode, N, t, name):
    w = configs.shrink(w, n_tokens=N, t=t)
    cache, wts = synth.make_cache(w, 0), synth.make_weights(w, 0)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, t)
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, t, mode=mode)
    assert_parity(got, ref, BF16_TOL if mode == configs.MODE_BF16 else FP32_TOL, name)


@pytest.mark.parametrize("mode", [configs.MODE_BF16, configs.MODE_FP32])
@pytest.mark.parametrize("scale", [0.173, 0.174])
def test_refinement_rule_edge(mode, scale):
    """Logit scales just below and just above the one (log2 e times it = 1/4)
    from which the near-maximal logits are recomputed."""
    w = configs.shrink(configs.get_workload(1), logit_scale_cross=scale)
    _layer_case(w, mode, 1000, 130, f"cfg1 scale {scale} mode {mode}")


def _attend_case(H, group, nq, t, S, d, causal, mode, rotate=False):
    import numpy as np
    import torch
    from oracle import consumer
    from paper_2606_07878_amd import binding
    from tests.helpers import dev_tensor, log, slice_errors
    a = synth.make_attend_inputs(7, H, group, nq, t, S, d, beta=t > 0)
    f = synth.as_f64(a)
    qpos = 5000.5 + np.arange(nq, dtype=np.float64) if rotate else None
    ref = consumer.attend(f["q"], f["C_k"], f["C_v"], None if a["beta"] is None else a["beta"].astype(np.float64),
                          f["K"], f["V"], group=group, causal=causal, q_positions=qpos, rope_theta=1e6)
    dv = {k: (dev_tensor(v, mode) if v is not None else None) for k, v in a.items()}
    out = binding.attend(dv["q"], dv["C_k"] if t else None, dv["C_v"] if t else None, dv["beta"] if t else None,
                         dv["K"] if S else None, dv["V"] if S else None, group=group, causal=causal,
                         q_positions=None if qpos is None else torch.from_numpy(qpos).cuda(), rope_theta=1e6)
    torch.cuda.synchronize()
    err = slice_errors(out.double().cpu().numpy(), ref).max()
    tol = 8e-3 if mode == configs.MODE_BF16 else 1e-5   # the bf16 output's rounding; fp32 sums
    log(f"attend H={H} group={group} nq={nq} t={t} S={S} d={d} causal={causal} mode={mode}: {err:.3e} (tol {tol:g})")
    assert err <= tol


@pytest.mark.parametrize("mode", [configs.MODE_BF16, configs.MODE_FP32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("group,nq,t,S,causal", [
    (2, 1, 700, 9, False),     # 2 rows: the decode kernel at every width
    (2, 2, 700, 5444, True),   # 4 rows over 2 x 6144 keys: decode kernel at widths 128 and 256
    (2, 2, 700, 5445, True),   # ... over one key more: matrix kernel
    (4, 2, 700, 324, True),    # 8 rows over 2 x 1024 keys: decode kernel at rows of 512 bytes and more
    (4, 2, 700, 325, True),    # ... over one key more: matrix kernel
    (5, 1, 0, 37, False),      # 5 rows, fewer keys than one chunk of most widths
    (1, 3, 0, 65, True),       # 3 rows without a compact part
    (3, 3, 31, 33, True),      # 9 rows in the 16-row tile; chunks of 32 cut short and spilling over by one
    (4, 4, 0, 16, True),       # 16 rows: the last; fewer keys than one chunk, most of them masked for the first row
    (1, 17, 129, 17, True),    # 17 rows: the first of the 32-row tile; five chunks, so one wave takes two
    (4, 8, 4500, 0, False),    # 32 rows: the last; several splits, no suffix
])
def test_attend_row_tiles(mode, d, group, nq, t, S, causal):
    _attend_case(2, group, nq, t, S, d, causal, mode, rotate=nq == 17)


@pytest.mark.parametrize("d,N,t", [
    (128, 1, 1), (128, 256, 128), (128, 257, 129),       # one block of 512 keys, partly past the padded keys
    (128, 512, 127), (128, 513, 130), (128, 769, 64),    # one whole block; one key into the second; past its half
    (128, 4700, 300),                                    # several key splits, the last one short
    (256, 255, 33), (256, 257, 129), (256, 1500, 260),   # blocks of 256 keys, 512 value features
])
def test_attention_blocks(d, N, t):
    w = configs.shrink(configs.get_workload(1), head_dim=d, n_kv_heads=2)
    _layer_case(w, configs.MODE_BF16, N, t, f"cfg1 d={d} N={N} t={t}")


def test_attention_candidates_of_equal_keys():
    """The same 100 tokens 41 times over (4100 keys): every latent's best key is
    there 41 times, and more near-maximal ones, over two splits' lists."""
    import numpy as np
    w = configs.shrink(configs.get_workload(1), head_dim=128, n_kv_heads=2, n_tokens=4100, t=40)
    base = synth.make_cache(w, 0, n_tokens=100)
    cache = dict(K=np.tile(base["K"], (1, 41, 1)), V=np.tile(base["V"], (1, 41, 1)),
                 positions=np.tile(base["positions"], 41))
    wts = synth.make_weights(w, 0)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, 40)
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, 40)
    assert_parity(got, ref, BF16_TOL, "41-fold keys")


@pytest.mark.parametrize("d,N,t", [(64, 65, 17), (128, 300, 33), (128, 40, 1), (256, 257, 15), (256, 700, 49)])
def test_fp64_refinement_tiles(d, N, t):
    """fp32 mode: candidate lists that fill 32-row (16-row at d = 256) tiles in part."""
    w = configs.shrink(configs.get_workload(1), head_dim=d, n_kv_heads=2)
    _layer_case(w, configs.MODE_FP32, N, t, f"cfg1 fp32 d={d} N={N} t={t}")


@pytest.mark.parametrize("N,t", [(1201, 67), (1204, 68), (520, 130)])
def test_backward_tiles(N, t):
    """8 KV heads, 8 cross heads of width 128: key-side products on 128 x 128
    tiles with a short last tile, attention-side operands with rows that are
    (1204, 68) and are not (1201, 67) 16-byte aligned, 64 x 64 tiles (520)."""
    from tests.test_gpu_backward import _grad_case
    w = configs.shrink(configs.get_workload(1), n_kv_heads=8, n_cross_heads=8)
    _grad_case(w, f"8 x 8 heads N={N} t={t}", N=N, t=t)


def test_values_of_a_head_past_4_gib():
    """6.1 million keys in one head of width 256: its values span 5.9 GiB.  The
    cache is one of 1024 tokens 6000 times over, which leaves the softmax
    average as it is; every value feature has an offset of its own."""
    import numpy as np
    import torch
    from paper_2606_07878_amd import binding
    from tests.helpers import dev_tensor, weights_to_device
    copies = 6000
    w = configs.shrink(configs.get_workload(1), head_dim=256, n_kv_heads=1, n_tokens=1024, t=24, logit_scale_cross=0.15)
    cache, wts = synth.make_cache(w, 0), synth.make_weights(w, 0)
    off = np.random.default_rng(3).normal(0.0, 3.0, (1, 1, 256))
    cache["V"] = synth.bf16_bits(synth.as_f64(cache)["V"] + off)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, w.t)
    K, V = (dev_tensor(cache[n], configs.MODE_BF16).repeat(1, copies, 1) for n in ("K", "V"))
    pos = torch.from_numpy(cache["positions"]).cuda().repeat(copies)
    W = weights_to_device(wts, configs.MODE_BF16)
    Ck, Cv, p = binding.compact_layer(w.cfg, W, K, V, pos, w.rope_theta, w.t)
    torch.cuda.synchronize()
    assert_parity((Ck.double().cpu().numpy(), Cv.double().cpu().numpy(), p.cpu().numpy()), ref, BF16_TOL,
                  "values past 4 GiB")


def _three_level_layer(levels, seed=5):
    """A one-block compactor with H = 2, nc = 8 and a cache in which the key
    n's logits lie about levels[n] log2 units below the largest, for every
    latent: the projections are a bias of two large components plus noise, and
    keys lean away from it by an angle that their level sets.  Keys rounded to
    fp16 move such a logit by some 0.1 log2 units, each by its own amount."""
    import numpy as np
    H, d, nc, dc, t, D = 2, 128, 8, 128, 1024, 128
    N = len(levels)
    w = configs.shrink(configs.get_workload(1), head_dim=d, n_kv_heads=H, n_tokens=N, t=t, latent_dim=D,
                       n_cross_heads=nc, n_self_heads=0, ffn_kind=configs.FFN_NONE, ffn_hidden=0,
                       logit_scale_cross=1024.0)
    r = np.random.default_rng(seed)
    wts = synth.make_weights(w, 0)
    e, g = np.zeros(dc), np.zeros(dc)
    e[[3, 5]], g[[20, 21]] = np.sqrt(0.5), np.sqrt(0.5)
    lean = np.sqrt(np.maximum(2 * np.asarray(levels) / (1024 * np.log2(np.e)), 0.0))   # 1 - cos = lean^2 / 2
    K = np.zeros((H, N, d))
    K[:, :, 0] = lean
    wk = r.normal(0.0, 1.5e-4, (nc, dc, 2 * d))
    wk[:, :, :d] = 0.0
    wk[:, :, 0] = g
    bits = synth.bf16_bits
    wts["b0.ca_wk"] = bits(wk.reshape(nc * dc, 2 * d))
    wq = r.normal(0.0, 1.5e-4, (nc, dc, D))
    wq[:, [3, 5]] = 0.0                         # the large components of q are exact in fp16
    wts["b0.ca_wq"] = bits(wq.reshape(nc * dc, D))
    wts["b0.ca_bq"] = wts["b0.ca_bk"] = bits(np.tile(e, nc))
    cache = dict(K=bits(K), V=bits(r.standard_normal((H, N, d))), positions=np.zeros(N))
    return w, cache, wts


def test_heaviest_keys_among_full_candidate_lists():
    """Sixteen keys carry the mass of every latent.  In their key split they
    come after many thousand keys that were candidates at the time and before
    some 3500 that stay within the refinement margin: neither may displace them."""
    import numpy as np
    N = 65536
    levels = np.full(N, 12.5)                   # below the margin once the heavy keys are seen
    levels[N - 3584:] = 9.6                     # within it
    levels[N - 3600:N - 3584] = 0.0             # the heavy keys
    w, cache, wts = _three_level_layer(levels)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, w.t, heads=[1])
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, w.t)
    assert_parity((got[0][1:], got[1][1:], got[2]), ref, BF16_TOL, "full candidate lists")


@pytest.mark.parametrize("scale", [0.2, 2.0, 30.0])
def test_logit_scales_that_fill_the_candidate_lists(scale):
    """Logit scales at which all keys (0.2, 2) or hundreds (30) lie within the
    refinement margin: lists of 1024 keys each are halved time and again."""
    w = configs.shrink(configs.get_workload(1), head_dim=128, n_kv_heads=2, n_tokens=16384, t=1024, n_cross_heads=8,
                       n_self_heads=0, logit_scale_cross=scale)
    cache, wts = synth.make_cache(w, 0), synth.make_weights(w, 0)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, w.t, heads=[1])
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, w.t)
    assert_parity((got[0][1:], got[1][1:], got[2]), ref, BF16_TOL, f"scale {scale}")


def test_negative_logit_scale_fp32():
    """fp32 mode at a scale of -1024: the near-maximal logits are recomputed as
    at +1024."""
    w = configs.shrink(configs.get_workload(1), logit_scale_cross=-1024.0)
    _layer_case(w, configs.MODE_FP32, 1000, 130, "scale -1024")


@pytest.mark.parametrize("t", [1, 33])
def test_full_candidate_lists_beside_padding_rows(t):
    """Lists that fill in lanes whose neighbours hold padding rows, which have no
    lists: 64 splits of 2048 keys, all within the refinement margin."""
    w = configs.shrink(configs.get_workload(1), head_dim=128, n_kv_heads=2, n_tokens=131072, t=t, n_cross_heads=8,
                       n_self_heads=0, logit_scale_cross=0.5)
    cache, wts = synth.make_cache(w, 0), synth.make_weights(w, 0)
    ref = run_oracle(w.cfg, cache, wts, w.rope_theta, t, heads=[1])
    got = run_gpu(w.cfg, cache, wts, w.rope_theta, t)
    assert_parity((got[0][1:], got[1][1:], got[2]), ref, BF16_TOL, f"padding rows t={t}")

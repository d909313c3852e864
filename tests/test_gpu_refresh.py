"""GPU parity of dasc_refresh against the fp64 oracle.

Bar: refreshed rows within 2e-3 of the oracle, measured per (request, head) as
max |got - want| / max |want| over the refreshed rows; every other row of the
active state bit-identical to its input.
"""

import math

import numpy as np
import pytest

import paper_2608_30386_amd as D
from paper_2608_30386_amd._lib import DASC_MAX_WINDOW
from oracle import pack as OK
from oracle import recurrence as OR
from tests.gpu_util import (announce, dev, dev_bf16, dev_i32, host_words, kimi_layer_oracle, plans,
                            restored_states, shape_of)
from workloads import WORKLOADS, bf16_bits_from_f32, log_lambda, refresh_inputs, states_host

pytestmark = pytest.mark.gpu

TOL = 2e-3


def run_refresh(sh, pool, layer, inv_row, inp, W, init="restored", slots=None, kernel=None):
    """dasc_refresh (or, with `kernel`, dasc_refresh_select on that kernel) on a copy of
    the pool; returns the pool after the call."""
    import torch

    n_req = inp["k"].shape[0]
    states = dev(pool)
    slots = list(range(n_req)) if slots is None else slots
    announce(f"refresh {sh} layer={layer} n_req={n_req} W={W} init={init} kernel={kernel}")
    args = (sh, layer, dev_i32(inv_row), states, dev_i32(slots), dev_bf16(inp["k"]),
            dev_bf16(inp["v"]), dev(inp["g"]), dev(inp["beta"]), W)
    if kernel is None:
        D.dasc_refresh(*args, init)
    else:
        D.dasc_refresh_select(*args, kernel, init)
    torch.cuda.synchronize()
    return states.cpu().numpy()


def check(sh, pool, got_pool, layer, inv_row, inp, pairs, init="restored", slots=None,
          oracle=None, report=None):
    """Refreshed rows vs the oracle on `pairs` (computed here, or given as `oracle` =
    (want, omitted)); all other rows bit-identical.  Returns the per-head max-normalised
    error; `report`, a dict, also receives the element-wise error (floor 1e-3 max|y|)."""
    n_req = inp["k"].shape[0]
    slots = list(range(n_req)) if slots is None else slots
    H, dk = sh.n_heads, sh.dk
    inv_layer = inv_row[layer * H * dk:(layer + 1) * H * dk]
    if oracle is None:
        layer_in = np.stack([pool[slots[n], layer] for n in range(n_req)])
        want, om = OR.refresh(layer_in, inv_layer, inp["k"], inp["v"], inp["g"], inp["beta"],
                              sh.n_qk_heads, init, pairs=pairs)
    else:
        want, om = oracle
    got = np.stack([got_pool[slots[n], layer, h] for n, h in pairs])
    err = OR.refresh_error(got, want, om, pairs)
    if report is not None:
        report["per_head"] = err
        report["elementwise"] = OR.refresh_error_elementwise(got, want, om, pairs)
        report["pairs"] = len(pairs)
    assert err <= TOL, f"refresh error {err:.3e} > {TOL}"
    # every row that is not refreshed keeps its bits, in every slot and layer
    mask = np.zeros(pool.shape[:4], dtype=bool)
    for n in range(n_req):
        mask[slots[n], layer] = om
    a = pool.view(np.uint32)[~mask]
    b = got_pool.view(np.uint32)[~mask]
    assert np.array_equal(a, b), "a row that is not omitted changed"
    return err


def sample_pairs(n_req, H, omitted, k, seed=0):
    rng = np.random.default_rng(seed)
    cand = [(n, h) for n in range(n_req) for h in range(H) if omitted[h].any()]
    idx = rng.choice(len(cand), size=min(k, len(cand)), replace=False)
    return [cand[i] for i in sorted(idx)]


@pytest.mark.parametrize("init", ["restored", "zero"])
def test_tiny_kda_all_heads(init):
    wl = WORKLOADS["tiny_kda"]
    lib, _ = plans(wl)
    sh = shape_of(wl)
    pool = restored_states(wl, lib, wl.n_req)
    inp = refresh_inputs(wl, 32, log_lambda(wl)[0])
    got = run_refresh(sh, pool, 0, lib["inv_row"], inp, 32, init)
    pairs = [(n, h) for n in range(wl.n_req) for h in range(wl.n_heads)]
    err = check(sh, pool, got, 0, lib["inv_row"], inp, pairs, init)
    announce(f"tiny_kda init={init} max rel err {err:.2e}")


@pytest.mark.parametrize("W", [256, 1024])
def test_kimi_layer_serving_shape_every_head(W):
    # every refreshed (request, head) of the serving shape (16 x 32 heads) against the fp64
    # oracle, in the launch the bench times
    wl, lib, pool, inp, pairs, want, om = kimi_layer_oracle(W)
    sh = shape_of(wl)
    got = run_refresh(sh, pool, 0, lib["inv_row"], inp, W)
    rep = {}
    err = check(sh, pool, got, 0, lib["inv_row"], inp, pairs, oracle=(want, om), report=rep)
    assert rep["pairs"] == wl.n_req * int(om.any(axis=1).sum())
    announce(f"kimi_layer W={W}: all {rep['pairs']} heads, max per-head rel err {err:.2e}, "
             f"element-wise {rep['elementwise']:.2e}")


def test_kimi_layer_serving_shape_w2048():
    wl = WORKLOADS["kimi_layer"]
    lib, _ = plans(wl)
    sh = shape_of(wl)
    W = 2048
    pool = restored_states(wl, lib, wl.n_req)
    inp = refresh_inputs(wl, W, log_lambda(wl)[0])
    got = run_refresh(sh, pool, 0, lib["inv_row"], inp, W)
    om = (lib["inv_row"] < 0).reshape(wl.n_heads, wl.dk)
    pairs = sample_pairs(wl.n_req, wl.n_heads, om, 64, seed=W)
    rep = {}
    err = check(sh, pool, got, 0, lib["inv_row"], inp, pairs, report=rep)
    announce(f"kimi_layer W={W}: {len(pairs)} sampled heads, max per-head rel err {err:.2e}, "
             f"element-wise {rep['elementwise']:.2e}")


def test_qwen_gdn_full_layers():
    # every omitted v-head of two whole layers (8 requests x 20 heads each) against the
    # fp64 oracle
    wl = WORKLOADS["qwen_gdn"]
    lib, _ = plans(wl)
    sh = shape_of(wl)
    n_req = wl.n_req
    pool = restored_states(wl, lib, n_req)
    lam = log_lambda(wl)
    for layer in (0, 35):
        inp = refresh_inputs(wl, 1024, lam[layer], salt=layer)
        got = run_refresh(sh, pool, layer, lib["inv_row"], inp, 1024)
        om = (lib["inv_row"][layer * 32 * 128:(layer + 1) * 32 * 128] < 0).reshape(32, 128)
        assert om.all(axis=1).sum() == 20                   # 20 of 32 v-heads omitted
        pairs = [(n, h) for n in range(n_req) for h in range(32) if om[h].any()]
        assert len(pairs) == 160
        rep = {}
        err = check(sh, pool, got, layer, lib["inv_row"], inp, pairs, report=rep)
        announce(f"qwen_gdn layer={layer}: all 160 heads, max per-head rel err {err:.2e}, "
                 f"element-wise {rep['elementwise']:.2e}")


@pytest.mark.parametrize("arch,dk,dv,H,Hqk,W", [
    ("kda", 32, 12, 3, 3, 1),
    ("kda", 64, 256, 2, 2, 33),
    ("kda", 128, 20, 2, 1, 100),
    ("gdn", 16, 64, 4, 2, 31),
    ("gdn", 128, 128, 4, 2, 65),
])
def test_ragged_shapes(arch, dk, dv, H, Hqk, W):
    rng = np.random.default_rng(dk * 1000 + dv + W)
    L, n_req = 2, 3
    sh = D.Shape(arch, L, H, Hqk, dk, dv)
    unit_shape = (L, H, dk) if arch == "kda" else (L, H)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=unit_shape))
    g_static[1, 0] = math.log(1e-3) / 2.0        # layer 1, head 0: every unit omitted
    g_static[1, 1] = math.log(1e-3) / 1e4        # layer 1, head 1: every unit kept
    plan = D.dasc_plan(sh, g_static, "threshold", 0, 64)
    n_pool = 5
    pool = (0.05 * rng.standard_normal((n_pool, L, H, dk, dv))).astype(np.float32)
    inv = plan["inv_row"]
    pool.reshape(n_pool, -1, dv)[:, inv < 0] = 0.0
    k = rng.standard_normal((n_req, Hqk, W, dk)).astype(np.float32)
    k /= np.linalg.norm(k, axis=-1, keepdims=True)
    gshape = (n_req, H, W, dk) if arch == "kda" else (n_req, H, W)
    lam = np.exp(rng.uniform(math.log(1e-3), 0, size=gshape[:2] + (1,) * (len(gshape) - 2)))
    inp = {
        "k": bf16_bits_from_f32(k),
        "v": bf16_bits_from_f32(rng.standard_normal((n_req, H, W, dv)).astype(np.float32)),
        "g": (-lam * np.logaddexp(0, rng.standard_normal(gshape))).astype(np.float32),
        "beta": (1 / (1 + np.exp(-rng.standard_normal((n_req, H, W))))).astype(np.float32),
    }
    slots = [4, 0, 2]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 1, inv, inp, W, init, slots=slots)
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        check(sh, pool, got, 1, inv, inp, pairs, init, slots=slots)


@pytest.mark.parametrize("arch,dk,dv,H,Hqk,W", [
    ("kda", 16, 4, 2, 2, 32), ("gdn", 16, 256, 2, 1, 33),       # one block of columns, all and one
    ("kda", 32, 64, 2, 2, 31), ("gdn", 32, 68, 4, 4, 64),       # 64 columns a block: exact, one over
    ("kda", 64, 36, 2, 2, 16), ("kda", 64, 32, 1, 1, 17),       # 32 a block; tiles of 16 tokens
    ("kda", 128, 16, 2, 2, 15), ("gdn", 128, 52, 2, 2, 48),     # 16 a block
])
def test_per_column_kernel_edges(arch, dk, dv, H, Hqk, W):
    # The per-column kernel at the edges of its column blocks (2048 / dk columns) and token
    # tiles (32 tokens up to dk = 32, else 16).  Everything is fp32, so a bound on rounding holds
    # here: about dk + 4 roundings per token of values of the size of the state, summed over
    # W tokens at worst linearly.
    L, n_req = 2, 3
    sh = D.Shape(arch, L, H, Hqk, dk, dv)
    rng = np.random.default_rng(dk + 7 * dv + W)
    unit_shape = (L, H, dk) if arch == "kda" else (L, H)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=unit_shape))
    g_static[1, 0] = math.log(1e-3) / 2.0
    inv = D.dasc_plan(sh, g_static, "threshold", 0, 64)["inv_row"]
    pool = (0.05 * rng.standard_normal((4, L, H, dk, dv))).astype(np.float32)
    k = rng.standard_normal((n_req, Hqk, W, dk)).astype(np.float32)
    k /= np.linalg.norm(k, axis=-1, keepdims=True)
    gshape = (n_req, H, W, dk) if arch == "kda" else (n_req, H, W)
    inp = {
        "k": bf16_bits_from_f32(k),
        "v": bf16_bits_from_f32(rng.standard_normal((n_req, H, W, dv)).astype(np.float32)),
        "g": (-0.3 * np.logaddexp(0, rng.standard_normal(gshape))).astype(np.float32),
        "beta": (1 / (1 + np.exp(-rng.standard_normal((n_req, H, W))))).astype(np.float32),
    }
    slots = [3, 0, 2]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 1, inv, inp, W, init, slots=slots)
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        err = check(sh, pool, got, 1, inv, inp, pairs, init, slots=slots)
        assert err <= W * (dk + 4) * 2.0 ** -24, err


def _inputs_128(arch, n_req, H, Hqk, W, seed, g_lo=None):
    rng = np.random.default_rng(seed)
    dk = dv = 128
    k = rng.standard_normal((n_req, Hqk, W, dk)).astype(np.float32)
    k /= np.linalg.norm(k, axis=-1, keepdims=True)
    gshape = (n_req, H, W, dk) if arch == "kda" else (n_req, H, W)
    lam = np.exp(rng.uniform(math.log(1e-4), 0, size=gshape[:2] + (1,) * (len(gshape) - 2)))
    g = -lam * np.logaddexp(0, rng.standard_normal(gshape))
    if g_lo is not None:        # plant very strong decays on a few tokens
        m = rng.random(gshape) < 0.05
        g = np.where(m, rng.uniform(g_lo, -8.0, size=gshape), g)
    return {
        "k": bf16_bits_from_f32(k),
        "v": bf16_bits_from_f32(rng.standard_normal((n_req, H, W, dv)).astype(np.float32)),
        "g": g.astype(np.float32),
        "beta": (1 / (1 + np.exp(-rng.standard_normal((n_req, H, W))))).astype(np.float32),
    }


@pytest.mark.parametrize("arch,W,g_lo", [
    ("kda", 1, None), ("kda", 31, None), ("kda", 33, None), ("kda", 100, None),
    ("kda", 64, -30.0), ("gdn", 1, None), ("gdn", 31, None), ("gdn", 33, None),
    ("gdn", 47, None), ("gdn", 63, None), ("gdn", 65, None), ("gdn", 96, -30.0),
    ("gdn", 129, None), ("gdn", 200, -30.0),
])
def test_chunked_kernel_ragged_and_strong_decay(arch, W, g_lo):
    # dk = dv = 128 takes the chunked MFMA kernel; ragged last chunks and very strong
    # decays (floored at -10 inside the kernel) must stay within the bar
    L, H, Hqk, n_req = 1, 4, 2, 3
    sh = D.Shape(arch, L, H, Hqk, 128, 128)
    rng = np.random.default_rng(W)
    unit_shape = (L, H, 128) if arch == "kda" else (L, H)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=unit_shape))
    g_static[0, 0] = math.log(1e-3) / 2.0
    plan = D.dasc_plan(sh, g_static, "threshold", 0, 64)
    inv = plan["inv_row"]
    pool = (0.05 * rng.standard_normal((4, L, H, 128, 128))).astype(np.float32)
    pool.reshape(4, -1, 128)[:, inv < 0] = 0.0
    inp = _inputs_128(arch, n_req, H, Hqk, W, seed=W, g_lo=g_lo)
    slots = [3, 1, 0]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 0, inv, inp, W, init, slots=slots)
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        err = check(sh, pool, got, 0, inv, inp, pairs, init, slots=slots)
        announce(f"chunked {arch} W={W} g_lo={g_lo} init={init} max rel err {err:.2e}")


@pytest.mark.parametrize("strong_chunks", [(0, 2, 3), (1, 4)])
def test_kda_fast_and_strong_chunks_interleaved(strong_chunks):
    # Chunks of 32 tokens where some channel decays by more than 2^96 take the
    # strong-decay path, the others the fast path, decided per chunk.  Here one channel of
    # every head decays at every token of the chosen chunks (log-gate -12, floored at -10
    # inside the kernel: 2^-461 over a chunk), so that the window switches paths at chosen
    # chunk boundaries, including the first chunk and the ragged last one (W = 150).
    L, H, Hqk, n_req, W = 1, 4, 2, 3, 150
    sh = D.Shape("kda", L, H, Hqk, 128, 128)
    rng = np.random.default_rng(7)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=(L, H, 128)))
    plan = D.dasc_plan(sh, g_static, "threshold", 0, 64)
    inv = plan["inv_row"]
    pool = (0.05 * rng.standard_normal((4, L, H, 128, 128))).astype(np.float32)
    pool.reshape(4, -1, 128)[:, inv < 0] = 0.0
    inp = _inputs_128("kda", n_req, H, Hqk, W, seed=11)
    for c in strong_chunks:
        inp["g"][:, :, 32 * c:32 * (c + 1), 5] = -12.0
    slots = [2, 0, 3]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 0, inv, inp, W, init, slots=slots)
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        err = check(sh, pool, got, 0, inv, inp, pairs, init, slots=slots)
        announce(f"strong chunks {strong_chunks} init={init} max rel err {err:.2e}")


@pytest.mark.parametrize("W,strong", [
    (32, ()), (64, (1,)), (65, (0, 2)), (96, (0,)), (127, (1, 3)), (161, (0, 1, 5)),
])
def test_kda_chunk_counts_and_strong_channel_groups(W, strong):
    # 1 to 6 chunks (the block works on three chunks at a time, so the first and last ones
    # run with part of its waves idle), and the strong-decay path taken by some groups of 32
    # channels and not by others: one channel of the second and one of the last group decay
    # by 2^-461 over each chosen chunk
    L, H, Hqk, n_req = 1, 3, 3, 2
    sh = D.Shape("kda", L, H, Hqk, 128, 128)
    rng = np.random.default_rng(W)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=(L, H, 128)))
    inv = D.dasc_plan(sh, g_static, "threshold", 0, 64)["inv_row"]
    pool = (0.05 * rng.standard_normal((3, L, H, 128, 128))).astype(np.float32)
    pool.reshape(3, -1, 128)[:, inv < 0] = 0.0
    inp = _inputs_128("kda", n_req, H, Hqk, W, seed=W + 1)
    for c in strong:
        inp["g"][:, :, 32 * c:32 * (c + 1), [40, 127]] = -12.0
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 0, inv, inp, W, init, slots=[2, 0])
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        err = check(sh, pool, got, 0, inv, inp, pairs, init, slots=[2, 0])
        announce(f"kda W={W} strong={strong} init={init} max rel err {err:.2e}")


@pytest.mark.parametrize("kernel", [None, "channel_wy"])
def test_gdn_fast_and_strong_chunks_interleaved(kernel):
    # The same switch with one gate per token (GDN heads): the chosen chunks decay at every
    # token, on the GDN kernel and on the channel-wise kernel with its scalar-gate loads.
    L, H, Hqk, n_req, W = 1, 4, 2, 3, 150
    sh = D.Shape("gdn", L, H, Hqk, 128, 128)
    rng = np.random.default_rng(8)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=(L, H)))
    g_static[0, 0] = math.log(1e-3) / 2.0
    plan = D.dasc_plan(sh, g_static, "threshold", 0, 64)
    inv = plan["inv_row"]
    pool = (0.05 * rng.standard_normal((4, L, H, 128, 128))).astype(np.float32)
    pool.reshape(4, -1, 128)[:, inv < 0] = 0.0
    inp = _inputs_128("gdn", n_req, H, Hqk, W, seed=12)
    for c in (0, 2, 3):
        inp["g"][:, 1:, 32 * c:32 * (c + 1)] = -12.0
    slots = [1, 3, 0]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 0, inv, inp, W, init, slots=slots, kernel=kernel)
        pairs = [(n, h) for n in range(n_req) for h in range(H)]
        err = check(sh, pool, got, 0, inv, inp, pairs, init, slots=slots)
        announce(f"gdn strong chunks kernel={kernel} init={init} max rel err {err:.2e}")


def test_chunked_and_column_kernels_agree():
    wl = WORKLOADS["kimi_layer"]
    lib, _ = plans(wl)
    sh = shape_of(wl)
    n_req = 4
    pool = restored_states(wl, lib, n_req)
    inp = refresh_inputs(wl, 160, log_lambda(wl)[0], n_req=n_req)
    a = run_refresh(sh, pool, 0, lib["inv_row"], inp, 160)
    b = run_refresh(sh, pool, 0, lib["inv_row"], inp, 160, kernel="column")
    om = lib["inv_row"] < 0
    diff = np.abs(a.reshape(n_req, -1, 128)[:, om] - b.reshape(n_req, -1, 128)[:, om]).max()
    scale = np.abs(b.reshape(n_req, -1, 128)[:, om]).max()
    announce(f"chunked vs column max diff / max {diff / scale:.2e}")
    assert diff <= 1e-3 * scale
    assert np.array_equal(a.reshape(n_req, -1, 128)[:, ~om], b.reshape(n_req, -1, 128)[:, ~om])


def test_gdn_scalar_gate_kernel_matches_channel_kernel():
    # GDN heads take the scalar-gate kernel; the channel-wise kernel must give the same
    # state to within both kernels' distance from the oracle, and both stay in the bar
    wl = WORKLOADS["qwen_gdn"]
    lib, _ = plans(wl)
    sh = shape_of(wl)
    n_req, layer, W = 3, 5, 333
    pool = restored_states(wl, lib, n_req)
    inp = refresh_inputs(wl, W, log_lambda(wl)[layer], n_req=n_req, salt=layer)
    a = run_refresh(sh, pool, layer, lib["inv_row"], inp, W)
    b = run_refresh(sh, pool, layer, lib["inv_row"], inp, W, kernel="channel_wy")
    lo = layer * sh.n_heads * sh.dk
    om = (lib["inv_row"][lo:lo + sh.n_heads * sh.dk] < 0).reshape(sh.n_heads, sh.dk)
    pairs = sample_pairs(n_req, sh.n_heads, om, 6, seed=1)
    for got in (a, b):
        check(sh, pool, got, layer, lib["inv_row"], inp, pairs)
    diff = np.abs(a[:, layer][:, om] - b[:, layer][:, om]).max()
    scale = np.abs(b[:, layer][:, om]).max()
    announce(f"gdn scalar-gate vs channel kernel max diff / max {diff / scale:.2e}")
    assert diff <= 1e-4 * scale


def test_gdn_workspace_reuse():
    # the caller's workspace is asked for and left untouched: one buffer, full of another
    # pattern and reused by calls with different windows, gives the bits of a freshly drawn one
    import torch

    L, H, Hqk, n_req = 1, 4, 2, 3
    sh = D.Shape("gdn", L, H, Hqk, 128, 128)
    rng = np.random.default_rng(11)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=(L, H)))
    g_static[0, 0] = math.log(1e-3) / 2.0
    g_static[0, 3] = math.log(1e-3) / 2.0
    inv = D.dasc_plan(sh, g_static, "threshold", 0, 64)["inv_row"]
    pool = (0.05 * rng.standard_normal((3, L, H, 128, 128))).astype(np.float32)
    pool.reshape(3, -1, 128)[:, inv < 0] = 0.0
    ws = torch.full((D.dasc_refresh_workspace_bytes(sh, n_req, 160),), 0x7F, dtype=torch.uint8,
                    device="cuda")
    for W in (160, 40):
        inp = _inputs_128("gdn", n_req, H, Hqk, W, seed=W)
        args = (dev_i32(inv), None, dev_i32([2, 0, 1]), dev_bf16(inp["k"]), dev_bf16(inp["v"]),
                dev(inp["g"]), dev(inp["beta"]), W)
        outs = []
        for workspace in (ws, None):
            states = dev(pool)
            announce(f"gdn workspace reuse W={W} explicit={workspace is not None}")
            D.dasc_refresh(sh, 0, args[0], states, *args[2:], workspace=workspace)
            torch.cuda.synchronize()
            outs.append(states.cpu().numpy())
        assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
        check(sh, pool, outs[0], 0, inv, inp, [(n, h) for n in range(n_req) for h in range(H)],
              slots=[2, 0, 1])
    assert bool((ws == 0x7F).all())


@pytest.mark.parametrize("arch", ["kda", "gdn"])
def test_maximum_window(arch):
    # W = DASC_MAX_WINDOW (2^21 tokens): every token but the last 1024 is an identity step
    # (k = v = 0, g = 0, beta = 0: no decay, no update, exactly), so the result is the
    # oracle's replay of those 1024 tokens from the restored state.  The kernels still walk
    # the whole window: 65,536 chunks, input offsets up to 2^30 bytes, a 512 MiB GDN
    # workspace.  GDN: two v-heads on one key head.
    import torch

    W, tail = DASC_MAX_WINDOW, 1024
    L, H, n_req = 1, 2, 1
    Hqk = 2 if arch == "kda" else 1
    sh = D.Shape(arch, L, H, Hqk, 128, 128)
    rng = np.random.default_rng(21)
    unit_shape = (L, H, 128) if arch == "kda" else (L, H)
    g_static = D.dasc_static_log_decay(rng.uniform(math.log(1e-4), 0, size=unit_shape))
    g_static[0, 0] = math.log(1e-3) / 2.0             # head 0 (GDN) / row 0 (KDA) omitted
    if arch == "gdn":
        g_static[0, 1] = math.log(1e-3) / 1000.0      # head 1 kept
    inv = D.dasc_plan(sh, g_static, "threshold", 0, 64)["inv_row"]
    pool = (0.05 * rng.standard_normal((1, L, H, 128, 128))).astype(np.float32)
    pool.reshape(1, -1, 128)[:, inv < 0] = 0.0
    inp = _inputs_128(arch, n_req, H, Hqk, tail, seed=W)

    def whole(x, bits=False):
        shape = list(x.shape)
        shape[2] = W
        t = torch.zeros(shape, dtype=torch.bfloat16 if bits else torch.float32, device="cuda")
        t[:, :, W - tail:] = dev_bf16(x) if bits else dev(x)
        return t

    k, v = whole(inp["k"], bits=True), whole(inp["v"], bits=True)
    g, beta = whole(inp["g"]), whole(inp["beta"])
    states = dev(pool)
    announce(f"refresh {sh} n_req=1 W={W} (identity steps but the last {tail})")
    D.dasc_refresh(sh, 0, dev_i32(inv), states, dev_i32([0]), k, v, g, beta, W)
    torch.cuda.synchronize()
    got = states.cpu().numpy()
    del k, v, g, beta
    om = (inv < 0).reshape(H, 128)
    pairs = [(0, h) for h in range(H) if om[h].any()]
    assert pairs
    err = check(sh, pool, got, 0, inv, inp, pairs)
    announce(f"maximum window {arch}: max rel err {err:.2e}")


# What the 128 x 128 kernels' arithmetic allows, as a share of a head's norm.  Splitting an operand
# into bf16 high and low parts (8 bits each) moves it by at most 2^-17, and a product of two drops
# the low parts' product; over many entries the root mean square of each of these three is below
# 2^-18 of its term (2.4e-6, 2.4e-6 and 2.6e-6).  Three products follow one another in a chunk.
# All nine added up:
SPLIT_BOUND = 3 * 3 * 2.0 ** -18


def norm_errors(sh, pool, got_pool, layer, inv, inp, pairs, slots):
    """Per pair: 2-norm of the refreshed rows' error over the 2-norm of the rows."""
    layer_in = np.stack([pool[s, layer] for s in slots])
    H, dk = sh.n_heads, sh.dk
    want, om = OR.refresh(layer_in, inv[layer * H * dk:(layer + 1) * H * dk], inp["k"], inp["v"],
                          inp["g"], inp["beta"], sh.n_qk_heads, "restored", pairs=pairs)
    errs = []
    for (n, h), w in zip(pairs, want):
        got = got_pool[slots[n], layer, h].astype(np.float64)
        errs.append(np.linalg.norm((got - w)[om[h]]) / np.linalg.norm(w[om[h]]))
    return np.array(errs)


def test_gdn_correlated_keys():
    # Keys of length 1.35 around one direction per key head, beta = 1, slow decays: the inverse
    # of a chunk's I + A has large entries that cancel in its block (1, 0), so that block must
    # not be formed from 16-bit operands.
    n_req, H, Hqk, W = 3, 8, 4, 96
    sh = D.Shape("gdn", 1, H, Hqk, 128, 128)
    rng = np.random.default_rng(0)
    inv = np.full(H * 128, -1, np.int32)
    pool = (0.05 * rng.standard_normal((n_req, 1, H, 128, 128))).astype(np.float32)
    inp = _inputs_128("gdn", n_req, H, Hqk, W, seed=1)
    k = 0.3 * rng.standard_normal((n_req, Hqk, W, 128)) + rng.standard_normal((n_req, Hqk, 1, 128))
    k *= 1.35 / np.linalg.norm(k, axis=-1, keepdims=True)
    inp["k"] = bf16_bits_from_f32(k.astype(np.float32))
    inp["beta"] = np.ones_like(inp["beta"])
    inp["g"] = (-1e-3 * np.logaddexp(0, rng.standard_normal((n_req, H, W)))).astype(np.float32)
    got = run_refresh(sh, pool, 0, inv, inp, W)
    pairs = [(n, h) for n in range(n_req) for h in range(H)]
    errs = norm_errors(sh, pool, got, 0, inv, inp, pairs, list(range(n_req)))
    announce(f"gdn correlated keys: error of the norm mean {errs.mean():.2e} max {errs.max():.2e}")
    assert errs.mean() <= SPLIT_BOUND


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("arch", ["kda", "gdn"])
def test_more_heads_than_one_grid_holds(arch, fused):
    # 7,536,640 heads: one block of 576 (KDA) or 640 (GDN) threads each would be more threads than
    # the 2^32 a grid may have.  All requests but the first and the last have a slot outside the
    # pool, which skips them; those two must come out as they do alone.
    import torch

    n_req, H, W = 1840, 4096, 1
    sh = D.Shape(arch, 1, H, 1, 128, 128)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def rand(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    live = [0, n_req - 1]
    inv = torch.arange(H * 128, dtype=torch.int32, device="cuda")
    inv = torch.where((inv // 128) % 64 == 5, -1, inv)         # 64 of the 4096 heads refreshed
    gs = (H, W, 128) if arch == "kda" else (H, W)
    k = torch.zeros((n_req, 1, W, 128), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros((n_req, H, W, 128), dtype=torch.bfloat16, device="cuda")
    g, beta = torch.zeros((n_req, *gs), device="cuda"), torch.zeros((n_req, H, W), device="cuda")
    for i in live:
        k[i] = (rand(1, W, 128) / 128 ** 0.5).to(torch.bfloat16)
        v[i] = rand(H, W, 128).to(torch.bfloat16)
        g[i], beta[i] = -rand(*gs).abs(), torch.sigmoid(rand(H, W))
    pool = 0.05 * rand(2, 1, H, 128, 128)
    ckpt = 0.05 * rand(2, H * 128, 128) if fused else None
    ws_bytes = D.dasc_refresh_workspace_bytes(sh, n_req, W)

    def call(states, slots, sel):
        ids = torch.as_tensor(slots, dtype=torch.int32, device="cuda")
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda") if ws_bytes else None
        a = (k[sel], v[sel], g[sel], beta[sel], W)
        announce(f"{'fused ' if fused else ''}refresh {sh} n_req={ids.numel()}")
        if fused:
            D.dasc_restore_refresh(sh, 0, ckpt, ids, inv, states, ids, *a, n_rows=H * 128, workspace=ws)
        else:
            D.dasc_refresh(sh, 0, inv, states, ids, *a, workspace=ws)
        torch.cuda.synchronize()
        return states

    slots = [-1] * n_req
    slots[0], slots[-1] = 0, 1
    got = call(pool.clone(), slots, slice(None))
    want = pool.clone()
    for s, i in enumerate(live):
        call(want, [s], slice(i, i + 1))
    assert not torch.equal(want, pool)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("arch,dk,dv", [
    ("kda", 16, 4), ("gdn", 16, 32), ("kda", 16, 36), ("gdn", 16, 64), ("kda", 16, 68),
    ("kda", 32, 16), ("gdn", 32, 20), ("kda", 32, 32), ("gdn", 32, 36),
])
def test_per_column_kernel_narrow_heads(arch, dk, dv):
    # From 512 heads on, heads of 16 or 32 rows take blocks of 64 or 128 threads if these hold all
    # their columns (dv * dk / 8 lanes).  A lane does the same whatever its block, so every request
    # must come out bit for bit as in a call of its own (which takes 256 threads); the first and
    # the last also against the oracle, within the rounding bound of the per-column kernel.
    n_req, H, W = 128, 4, 35
    sh = D.Shape(arch, 1, H, H, dk, dv)
    rng = np.random.default_rng(dk + dv)
    inv = rng.integers(-1, 1, size=(H, dk)) if arch == "kda" else np.full((H, dk), -1)
    inv[1] = 0                                              # head 1 kept
    inv = inv.astype(np.int32).reshape(-1)
    pool = (0.05 * rng.standard_normal((n_req, 1, H, dk, dv))).astype(np.float32)
    k = rng.standard_normal((n_req, H, W, dk)).astype(np.float32)
    k /= np.linalg.norm(k, axis=-1, keepdims=True)
    gshape = (n_req, H, W, dk) if arch == "kda" else (n_req, H, W)
    inp = {
        "k": bf16_bits_from_f32(k),
        "v": bf16_bits_from_f32(rng.standard_normal((n_req, H, W, dv)).astype(np.float32)),
        "g": (-0.3 * np.logaddexp(0, rng.standard_normal(gshape))).astype(np.float32),
        "beta": (1 / (1 + np.exp(-rng.standard_normal((n_req, H, W))))).astype(np.float32),
    }
    got = run_refresh(sh, pool, 0, inv, inp, W)
    for n in range(0, n_req, 9):
        one = run_refresh(sh, pool[n:n + 1], 0, inv, {x: a[n:n + 1] for x, a in inp.items()}, W)
        assert np.array_equal(one[0].view(np.uint32), got[n].view(np.uint32)), n
    err = check(sh, pool, got, 0, inv, inp, [(n, h) for n in (0, n_req - 1) for h in range(H)])
    assert err <= W * (dk + 4) * 2.0 ** -24, err


@pytest.mark.parametrize("H,n_req,keep", [
    (32, 9, "some"), (32, 12, "some"), (64, 6, "some"), (64, 5, "none"), (5, 60, "some"),
    (1, 300, "none"), (1, 300, "all"), (7, 54, "rows"), (33, 8, "rows"), (65, 5, "some"),
])
def test_gdn_refreshed_heads_first(H, n_req, keep):
    # 257 to 384 heads of at most 64 a layer are dealt to the blocks with the refreshed ones first,
    # a head's first row standing for it; every request must come out bit for bit as in a call of
    # few heads.  keep: some heads, none, all, or single rows (also the first of a refreshed head,
    # or all but the first of one that then counts as refreshed by it alone).
    W = 40
    sh = D.Shape("gdn", 1, H, 1, 128, 128)
    assert 256 < n_req * H <= 384
    rng = np.random.default_rng(H + n_req)
    inv = np.full((H, 128), -1, np.int32)
    if keep == "all":
        inv[:] = 0
    elif keep == "some":
        inv[rng.permutation(H)[:max(1, 3 * H // 8)]] = 0
    elif keep == "rows":
        inv[0, 0] = 0
        inv[1, 1:] = 0
        inv[2:, :] = rng.integers(-1, 1, size=(H - 2, 128))
        inv[3] = 0
    inv = inv.reshape(-1)
    pool = (0.05 * rng.standard_normal((n_req, 1, H, 128, 128))).astype(np.float32)
    inp = _inputs_128("gdn", n_req, H, 1, W, seed=H)
    got = run_refresh(sh, pool, 0, inv, inp, W)
    step = max(1, 128 // H)
    for n in range(0, n_req, step):
        part = {x: a[n:n + step] for x, a in inp.items()}
        few = run_refresh(sh, pool[n:n + step], 0, inv, part, W)
        assert np.array_equal(few.view(np.uint32), got[n:n + step].view(np.uint32)), n
    if keep != "all":
        om = (inv < 0).reshape(H, 128)
        heads = [h for h in range(H) if om[h].any()]
        check(sh, pool, got, 0, inv, inp, [(n_req - 1, h) for h in (heads[0], heads[-1])])


# log2 decays over each chunk of 32 tokens (the last one repeats), by group of 32 channels
LAGS = {
    "steady": ([5.0], [19.0], [39.0], [60.0]),          # applied at the end, every 3rd, 2nd, 1st chunk
    "at the bound": ([13.3], [13.4], [20.0], [20.1]),   # 3 x 13.4 and 2 x 20.1 pass 40, the others not
    "crossing": ([39.0, 60.0, 39.0], [200.0, 5.0], [5.0, 5.0, 200.0, 3.0], [30.0, 90.0, 30.0]),
    "mixed": ([0.01], [39.9, 0.2], [10.0, 150.0, 10.0], [96.0, 1.0]),
    "slow": ([0.1], [0.5], [1.0], [2.0]),               # carried to the end, most of the state kept
}
# the same by head for GDN, whose state may lag by 2^16
GDN_LAGS = {
    "steady": ([0.1], [1.0], [5.0], [60.0]),
    "at the bound": ([5.3], [5.4], [8.0], [8.1]),
    "mixed": ([15.9, 0.2], [4.0, 150.0, 4.0], [0.01], [300.0, 1.0, 15.5, 1.0]),
}


@pytest.mark.parametrize("W", [96, 201])
@pytest.mark.parametrize("lags", LAGS)
def test_kda_state_decay_carried_over_chunks(lags, W):
    # The kernel multiplies the decay of 32 channels into the state only when it has lagged by 2^40:
    # lags of several chunks, just below and above the bound, groups of one head that apply it in
    # different chunks, a lag that takes a chunk past 2^96 onto the strong-decay path, and lags
    # that follow or precede a chunk on it.  Each group of rows on its own, against what the split
    # products allow, and the exponents: a running sum near 2^7 is within 2^-17 of its value, the
    # decay then within 2^-17 ln 2.
    n_req, H = 2, 3
    sh = D.Shape("kda", 1, H, H, 128, 128)
    rng = np.random.default_rng(W)
    inv = np.full(H * 128, -1, np.int32)
    pool = (0.05 * rng.standard_normal((n_req, 1, H, 128, 128))).astype(np.float32)
    inp = _inputs_128("kda", n_req, H, H, W, seed=W + 2)
    g = np.empty((W, 128))
    for grp, per_chunk in enumerate(LAGS[lags]):
        for t in range(W):
            g[t, 32 * grp:32 * grp + 32] = -per_chunk[min(t // 32, len(per_chunk) - 1)] * math.log(2) / 32
    inp["g"] = np.broadcast_to(g, (n_req, H, W, 128)).astype(np.float32)
    pairs = [(n, h) for n in range(n_req) for h in range(H)]
    for init in ("restored", "zero"):
        got = run_refresh(sh, pool, 0, inv, inp, W, init)
        want, _ = OR.refresh(pool[:, 0], inv, inp["k"], inp["v"], inp["g"], inp["beta"], H, init,
                             pairs=pairs)
        have = np.stack([got[n, 0, h] for n, h in pairs]).astype(np.float64)
        d = (have - want).reshape(len(pairs), 4, -1)
        err = np.linalg.norm(d, axis=-1) / np.linalg.norm(want.reshape(len(pairs), 4, -1), axis=-1)
        announce(f"lags {lags} W={W} init={init}: error by group {[f'{e:.1e}' for e in err.max(axis=0)]}")
        assert err.max() <= SPLIT_BOUND + 2.0 ** -17 * math.log(2)


@pytest.mark.parametrize("n_req", [2, 33])
@pytest.mark.parametrize("lags", GDN_LAGS)
def test_gdn_state_decay_carried_over_chunks(lags, n_req):
    # As above for GDN heads, four rates in the four heads of a request, with two blocks per head
    # (8 heads) and with one (132).
    H, W = 4, 201
    sh = D.Shape("gdn", 1, H, 2, 128, 128)
    rng = np.random.default_rng(n_req)
    inv = np.full(H * 128, -1, np.int32)
    pool = (0.05 * rng.standard_normal((n_req, 1, H, 128, 128))).astype(np.float32)
    inp = _inputs_128("gdn", n_req, H, 2, W, seed=n_req + 2)
    for h, per_chunk in enumerate(GDN_LAGS[lags]):
        for t in range(W):
            inp["g"][:, h, t] = -per_chunk[min(t // 32, len(per_chunk) - 1)] * math.log(2) / 32
    pairs = [(n, h) for n in (0, n_req - 1) for h in range(H)]
    got = run_refresh(sh, pool, 0, inv, inp, W)
    errs = norm_errors(sh, pool, got, 0, inv, inp, pairs, list(range(n_req)))
    announce(f"gdn lags {lags} n_req={n_req}: error {[f'{e:.1e}' for e in errs]}")
    assert errs.max() <= SPLIT_BOUND + 2.0 ** -17 * math.log(2)


def test_gdn_update_scale_keeps_exact_betas():
    # One chunk from a zero state with the unit vectors as keys: T is the identity, so row t of the
    # state is 2^{..} beta_t v_t.  With betas that bf16 holds, T' and U are exact and the only
    # rounding above fp32's is the split of the scaled U: the high part leaves at most half its last
    # place, 2^-8 of the power of two below, the low part 2^-9 of that, so at most 2^-17 of each
    # entry.  Exponents below 2 and the exponential add less than 2^-21.  Rounding T' too would
    # double it.
    n_req, H, W = 2, 4, 32
    sh = D.Shape("gdn", 1, H, H, 128, 128)
    rng = np.random.default_rng(4)
    inv = np.full(H * 128, -1, np.int32)
    pool = np.zeros((n_req, 1, H, 128, 128), np.float32)
    inp = _inputs_128("gdn", n_req, H, H, W, seed=4)
    inp["k"] = bf16_bits_from_f32(np.broadcast_to(np.eye(W, 128, dtype=np.float32), (n_req, H, W, 128)).copy())
    inp["beta"] = rng.choice([0.25, 0.5, 1.0], size=(n_req, H, W)).astype(np.float32)
    inp["g"] = (-0.04 * rng.random((n_req, H, W))).astype(np.float32)
    got = run_refresh(sh, pool, 0, inv, inp, W, "zero")
    pairs = [(n, h) for n in range(n_req) for h in range(H)]
    want, _ = OR.refresh(pool[:, 0], inv, inp["k"], inp["v"], inp["g"], inp["beta"], H, "zero", pairs=pairs)
    want = np.stack(want)[:, :W]
    err = np.abs(got[:, 0].reshape(-1, 128, 128)[:, :W] - want) / np.abs(want)
    announce(f"gdn unit keys, exact betas: largest relative error of an entry {err.max():.2e}")
    assert err.max() <= 2.0 ** -17 + 2.0 ** -21

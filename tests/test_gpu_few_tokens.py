"""Kernels that serve few tokens: the router split over experts, the one-workgroup index build (T <= 1024), the combine with a workgroup per token,
and the router backward in quarter tiles."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_05296_amd import binding as B
from paper_2601_05296_amd import layer, synth
from tests.parity import assert_close, dev, host, launched, near_tie_ok

pytestmark = pytest.mark.gpu


def _bf16(rng, shape, std):
    s = synth.bf16_round(rng.standard_normal(shape, dtype=np.float32) * np.float32(std))
    return s, synth.bf16_to_f32(s)


def _route(xs, ws, bias, T, d, E, k, renorm, want_logits=True):
    ids = torch.empty((T, k), dtype=torch.int32, device="cuda")
    gates = torch.empty((T, k), dtype=torch.float32, device="cuda")
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda") if want_logits else None
    B.moe_route(dev(xs), dev(ws), dev(bias), T, d, E, k, B.MOE_RENORM if renorm else 0, ids, gates,
                logits)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), host(gates), host(logits) if want_logits else None


# both sides of the split's bounds (E * d >= 65536, d >= 2 E; 16 tokens up to 32
# experts, 256 tiles up to 64, T * E <= 98304 beyond), ragged token and expert blocks,
# K shares of one to several steps
@pytest.mark.parametrize("T,d,E,k,renorm", [
    (1, 1024, 64, 6, True), (17, 4096, 16, 16, False), (100, 1984, 33, 3, False),
    (384, 256, 256, 16, True), (385, 256, 256, 16, True), (50, 320, 205, 8, False),
    (50, 320, 204, 8, False), (50, 512, 256, 16, False), (16, 4096, 16, 2, False),
    (1360, 2048, 33, 5, True), (1361, 2048, 33, 5, True), (768, 768, 128, 8, True),
    (769, 768, 128, 8, True)])
def test_route_few_tokens(T, d, E, k, renorm):
    rng = np.random.Generator(np.random.PCG64(T + E))
    xs, x = _bf16(rng, (T, d), 1.0)
    ws, wg = _bf16(rng, (E, d), 0.02)
    bias = rng.standard_normal(E, dtype=np.float32)
    bias[rng.integers(E)] = -np.inf
    ids_r, gates_r, logits_r, _ = oracle.route(x, wg, bias, k, renorm)
    ids, gates, logits = _route(xs, ws, bias, T, d, E, k, renorm)
    fin = np.isfinite(logits_r)
    assert np.array_equal(np.isfinite(logits), fin)
    assert_close("logits", logits[fin], logits_r[fin], "f32")
    assert near_tie_ok(ids, ids_r, np.where(fin, logits_r, -1e30)) <= 1
    same = np.all(ids == ids_r, axis=1)
    assert_close("gates", gates[same], gates_r[same], "f32")


# one and two K groups (odd slice counts and E > 128 have one), K shares that end
# in the middle of a wave's turn and of the last wave's, several rounds of turns
@pytest.mark.parametrize("T,d,E,k,renorm", [
    (1, 2048, 64, 6, True), (48, 2048, 64, 6, False), (300, 2880, 128, 4, False),
    (16, 4096, 16, 16, False), (9, 8320, 8, 2, False), (64, 1024, 200, 9, False),
    (70, 576, 130, 5, False), (40, 640, 103, 8, True), (21, 4160, 65, 3, False),
    (1024, 1088, 64, 6, False)])
def test_route_same_bits_in_one_and_two_launches(T, d, E, k, renorm):
    """A token's routing does not depend on the launches that compute it: without the
    logits output (one launch), and among so many tokens that one launch serves
    them, ids, gates and logits are the same bits."""
    rng = np.random.Generator(np.random.PCG64(T + d))
    xs, _ = _bf16(rng, (T, d), 1.0)
    ws, _ = _bf16(rng, (E, d), 0.02)
    bias = rng.standard_normal(E, dtype=np.float32)
    n = 98304 // (T * E) + 1
    assert n * T < 32768       # beyond, the one-launch router has one K group
    out = []

    def run(xs, T, want_logits):
        return launched(lambda: out.append(_route(xs, ws, bias, T, d, E, k, renorm, want_logits)))

    assert run(xs, T, True) == ["route_logits", "route_pick"]
    assert run(xs, T, False) == ["route_bf16"]
    assert run(np.tile(xs, (n, 1)), n * T, True) == ["route_bf16"]
    for a, b, c in zip(*out):
        assert b is None or np.array_equal(a, b)
        assert np.array_equal(a, c[:T])


def test_route_few_tokens_ties_and_nan():
    """Equal logits go to the lower id; NaN logits are never chosen (as in the
    one-launch router), and places without an expert get an id that the index
    build rejects."""
    E, k, T, d = 130, 4, 40, 512
    x = np.zeros((T, d), dtype=np.uint16)
    x[3] = 0x7FC0                                   # token 3: every logit NaN
    ws = np.zeros((E, d), dtype=np.uint16)
    bias = np.zeros(E, dtype=np.float32)
    bias[[7, 129]] = 1.0
    bias[[0, 5]] = np.nan
    ids, _, _ = _route(x, ws, bias, T, d, E, k, False)
    for t in range(T):
        if t == 3:
            assert np.all(ids[t] == 0x7FFFFFFF)
        else:
            assert ids[t].tolist() == [7, 129, 1, 2]


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (63, 5, 4), (64, 256, 16), (65, 64, 5), (1023, 128, 8),
                                   (1024, 200, 9), (1025, 200, 9)])
def test_index_one_workgroup(T, E, k):
    rng = np.random.Generator(np.random.PCG64(T))
    ids = synth.random_ids(T, E, k, seed=T)
    bad = rng.random(ids.shape) < 0.1               # rejected: out of range or a repeat
    ids[bad] = rng.choice([-1, E, 0x7FFFFFFF, 0], size=int(bad.sum()))
    rej = np.zeros(ids.shape, bool)
    for j in range(k):
        e = ids[:, j:j + 1]
        rej[:, j] = ((e < 0) | (e >= E))[:, 0] | (ids[:, :j] == e).any(1)
    ref = oracle.build_index(np.where(rej, E, ids), E + 1)
    i32 = dict(dtype=torch.int32, device="cuda")
    m = [torch.empty(n, **i32) for n in (E, E + 1, T * k, T * k, T * k)]
    n = B.moe_build_index_workspace_size(T, E, k)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    B.moe_build_index(dev(ids), T, E, k, *m, ws, n)
    torch.cuda.synchronize()
    counts, offsets, eti, tim, ss = (t.cpu().numpy() for t in m)
    f = int(ref.offsets[E])
    assert np.array_equal(counts, ref.counts[:E]) and np.array_equal(offsets, ref.offsets[:E + 1])
    assert np.array_equal(eti[:f], ref.eti[:f]) and np.array_equal(ss[:f], ref.slot_src[:f])
    assert np.array_equal(tim.reshape(T, k), np.where(rej, -1, ref.tim))


def test_clear_runs_at_the_fill_rate():
    """The atomic combine clears y and dx (268 MB here) as fast as a plain fill writes
    them: measured at 0.94 of the time of torch's zero_, a loop over 2048 workgroups
    at 1.16."""
    T, d, f, E, k = 32768, 4096, 64, 2, 1
    x, w1, w2 = (torch.randn(s, device="cuda").to(torch.bfloat16) for s in ((T, d), (E, d, f), (E, f, d)))
    wg = torch.randn((E, d), device="cuda").to(torch.bfloat16)
    times = {"fwd_prep": [], "zero_bf16": [], "fill": []}
    fill = torch.empty_like(x)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for _ in range(15):
        ev[0].record()
        fill.zero_()
        ev[1].record()
        torch.cuda.synchronize()
        times["fill"].append(ev[0].elapsed_time(ev[1]))
        B.moe_probe_enable(64)
        y, saved = layer.forward(x, wg, None, w1, None, w2, k, False, act="relu")
        layer.backward(saved, x, x, wg, w1, None, w2)
        torch.cuda.synchronize()
        for i in range(B.moe_probe_count()):
            name, ms = B.moe_probe_get(i)
            times.get(name, []).append(ms)
        B.moe_probe_disable()
    med = {n: float(np.median(t)) for n, t in times.items()}
    assert len(times["fwd_prep"]) == len(times["zero_bf16"]) == 15
    assert max(med["fwd_prep"], med["zero_bf16"]) <= 1.05 * med["fill"], med


# the last workgroup of each preparation launch: a clear longer and shorter than the
# slots, more of both than one grid of 2048 x 256 threads
@pytest.mark.parametrize("T,d,E,k", [(1, 64, 3, 1), (37, 64, 20, 16), (33, 64, 4, 2), (300001, 64, 2, 2),
                                     (21000, 1024, 2, 1)])
def test_clear_and_slot_gates(T, d, E, k):
    """The atomic combine with zero experts clears every row of y and leaves the gates
    in slot order in its workspace."""
    z = dict(dtype=torch.bfloat16, device="cuda")
    x = torch.randn((T, d), device="cuda").to(torch.bfloat16)
    ids = dev(synth.random_ids(T, E, k, seed=T))
    S, f, fl = T * k, 64, B.MOE_ACT_RELU | B.MOE_H_ON_LOAD | B.MOE_ATOMIC_COMBINE
    i32 = dict(dtype=torch.int32, device="cuda")
    m = [torch.empty(n, **i32) for n in (E, E + 1, S, S, S)]
    n = B.moe_build_index_workspace_size(T, E, k)
    B.moe_build_index(ids, T, E, k, *m, torch.empty(max(n, 16), dtype=torch.uint8, device="cuda"), n)
    gates = torch.rand((T, k), device="cuda")
    w1, w2 = torch.zeros((E, d, f), **z), torch.zeros((E, f, d), **z)
    y = torch.full((T, d), float("nan"), **z)
    A = torch.empty((S, f), **z)
    n = B.moe_ffn_fwd_combine_workspace_size(T, d, f, E, k, fl)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    B.moe_ffn_fwd_combine(x, w1, None, w2, m[1], m[2], gates, m[3], T, d, f, E, k, fl, A, None, y, ws, n)
    torch.cuda.synchronize()
    assert not y.any()
    # the workspace starts with the gates in slot order
    gs = ws[:4 * S].view(torch.float32)
    assert torch.equal(gs, gates.view(-1)[m[4].long()])

"""The row-wise GEMMs for few rows per expert return the bits of the 256-row
kernels: the same tokens, once alone (few rows per expert) and once repeated so
often that the 256-row kernels run, give equal A, B, O, dA, dB, dX_slot,
d_gates, y and dx. Expert loads sit on the edges of the 32-, 64- and 128-row
tiles; d and f are odd multiples of 64 (half-empty column tiles)."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_05296_amd import binding as B
from tests.parity import dev, launched

pytestmark = pytest.mark.gpu


def _bf16(rng, shape, std):
    t = torch.from_numpy(rng.standard_normal(size=shape, dtype=np.float32) * np.float32(std))
    return t.to(torch.bfloat16).cuda()


def _ffn(ids, gates, x, dy, w, act, h_on_load, atomic):
    """Forward and backward of the FFN calls on ids [T, 1]; slot order is
    expert by expert, ascending token."""
    w1, w3, w2 = w
    T, k = ids.shape
    E, d, f = w1.shape
    ix = oracle.build_index(ids, E)
    offsets, eti, tim, ss = (dev(a) for a in (ix.offsets, ix.eti, ix.tim, ix.slot_src))
    S = T * k
    gated = act == "swiglu"
    flags = B.ACT_FLAG[act] | (B.MOE_H_ON_LOAD if h_on_load else 0)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    A = torch.empty((S, f), **bf)
    Bm = torch.empty((S, f), **bf) if gated else None
    dw1, dw2 = torch.empty((E, d, f), **f32), torch.empty((E, f, d), **f32)
    dw3 = torch.empty((E, d, f), **f32) if gated else None
    dg = torch.empty((T, k), **f32)
    w3g = w3 if gated else None

    def ws(n):
        return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")

    out = {}
    if atomic:
        cf = flags | B.MOE_ATOMIC_COMBINE
        y, dx = torch.empty((T, d), **bf), torch.empty((T, d), **bf)
        n = B.moe_ffn_fwd_combine_workspace_size(T, d, f, E, k, cf)
        B.moe_ffn_fwd_combine(x, w1, w3g, w2, offsets, eti, gates, tim, T, d, f, E, k, cf, A, Bm,
                              y, ws(n), n)
        out.update(A=A.clone(), y=y)
        n = B.moe_ffn_bwd_combine_workspace_size(T, d, f, E, k, cf)
        B.moe_ffn_bwd_combine(dy, x, w1, w3g, w2, gates, offsets, eti, ss, tim, A, Bm, T, d, f, E,
                              k, cf, dw1, dw3, dw2, dg, dx, ws(n), n)
        out.update(dx=dx)
        rows = {"A": 1, "dA": 1}
    else:
        O, dX = torch.empty((S, d), **bf), torch.empty((S, d), **bf)
        n = B.moe_ffn_fwd_workspace_size(T, d, f, E, k, flags)
        B.moe_ffn_fwd(x, w1, w3g, w2, offsets, eti, T, d, f, E, k, flags, A, Bm, O, ws(n), n)
        out.update(A=A.clone(), O=O)
        if gated:
            out["B"] = Bm.clone()
        n = B.moe_ffn_bwd_workspace_size(T, d, f, E, k, flags)
        B.moe_ffn_bwd(dy, x, w1, w3g, w2, gates, offsets, eti, ss, A, Bm, T, d, f, E, k, flags,
                      dw1, dw3, dw2, dg, dX, ws(n), n)
        out.update(dX=dX)
        if gated:
            out["dB"] = Bm
    out.update(dA=A, dg=dg)
    torch.cuda.synchronize()
    # slot-ordered arrays back to token order
    order = torch.from_numpy(ix.tim[:, 0].astype(np.int64)).cuda()
    return {n: t if n in ("y", "dx", "dg") else t[order] for n, t in out.items()}


EDGES_64 = [1, 31, 32, 33, 63, 64, 65, 0]              # mean 36: 64-row tiles
EDGES_128 = [97, 127, 128, 129, 1, 64, 65, 100]        # mean 88: 128-row tiles


@pytest.mark.parametrize("counts,d,f,act,h_on_load,atomic", [
    ([3, 0, 0, 1, 0, 0, 2, 0], 192, 320, "swiglu", True, False),     # a few rows, slim tiles
    (EDGES_64, 192, 320, "swiglu", True, False),
    (EDGES_64, 320, 192, "swiglu", False, True),
    (EDGES_64, 128, 704, "relu", True, True),
    (EDGES_128, 192, 320, "swiglu", False, False),
    (EDGES_128, 320, 448, "silu", True, True),
    # enough experts for the wide tiles, forward and backward
    (EDGES_64 * 8, 192, 320, "swiglu", True, False),
    (EDGES_64 * 24, 576, 576, "silu", False, True),
    (EDGES_128 * 12, 576, 576, "swiglu", False, False),
    (EDGES_128 * 12, 64, 64, "swiglu", True, True),
    # many rows of few experts: launches that leave CUs idle in the large tiles
    ([700, 513], 320, 576, "swiglu", True, False),
    ([2049, 1, 1500], 192, 704, "silu", False, False),
    # ... h on load in 64 x 512 tiles, dX in 128-row tiles
    ([6000, 5000], 448, 192, "relu", True, True), ([6000, 5000], 448, 192, "swiglu", True, False),
    ([9000, 4100], 64, 128, "silu", True, True), ([9000, 4100], 64, 128, "silu", True, False),
    ([9000, 4100], 64, 128, "relu", True, False), ([9000, 4100], 64, 128, "swiglu", True, True)] + [
    # h formed on load in 32-row tiles of 128 and of 256 columns and in 64-row tiles of
    # 128 and of 256
    ([n] * E, d, 128, act, True, atomic)
    for E, n, d in ((24, 20, 768), (40, 20, 832), (24, 29, 768), (40, 29, 832))
    for act in ("swiglu", "silu", "relu") for atomic in (False, True)])
def test_small_rows_same_bits(counts, d, f, act, h_on_load, atomic):
    E, T = len(counts), sum(counts)
    rng = np.random.Generator(np.random.PCG64(T + d + f))
    ids = rng.permutation(np.repeat(np.arange(E), counts)).astype(np.int32)[:, None]
    x, dy = _bf16(rng, (T, d), 1.0), _bf16(rng, (T, d), 1.0)
    w = (_bf16(rng, (E, d, f), d ** -0.5), _bf16(rng, (E, d, f), d ** -0.5),
         _bf16(rng, (E, f, d), f ** -0.5))
    gates = torch.from_numpy(rng.random((T, 1), dtype=np.float32)).cuda()
    one, rep = {}, {}
    few = launched(lambda: one.update(_ffn(ids, gates, x, dy, w, act, h_on_load, atomic)))
    # repeats for a mean of 300 rows per expert and 130 row tiles of 256, beyond
    # every rule of the small kernels
    n = -(-max(300 * E, 130 * 256) // T)
    many = launched(lambda: rep.update(_ffn(np.tile(ids, (n, 1)), gates.repeat(n, 1),
                                            x.repeat(n, 1), dy.repeat(n, 1), w, act, h_on_load,
                                            atomic)))
    # the two runs take different kernels in every row-wise GEMM: G1, the second, G4, dX
    # (G1 of 6000 and 5000 rows in 64 + 64 columns has too many tiles for the small ones)
    gemms = ("g1", "g2", "g2h", "g4", "g6")
    few = [k for k in few if k.replace("sk_", "").split("_")[0] in gemms]
    many = [k for k in many if k.replace("sk_", "").split("_")[0] in gemms]
    assert many == ["g1_kernel", "g2h_kernel" if h_on_load else "g2_kernel", "g4_kernel", "g6_kernel"]
    second = ("sk_g2h", "g2h_narrow") if h_on_load else ("sk_g2",)
    assert few[1] in second and few[2:] == ["sk_g4", "sk_g6"], few
    if max(counts) > 4000:
        assert few[1] == "g2h_narrow"
    elif len(set(counts)) == 1:
        assert few[1] == "sk_g2h"
    assert few[0] == "sk_g1" or (act == "swiglu" and max(counts) == 6000), few
    for name, a in one.items():
        assert torch.isfinite(a.float()).all(), name
        assert torch.equal(a, rep[name][:T]), name
        assert torch.equal(a, rep[name][-T:]), name


@pytest.mark.parametrize("E,rows,d,f,act,h_on_load", [
    # full and partial tiles of the large weight-gradient tiles (more than 128 of
    # them, more than 96 slots per expert), and of the small ones
    (40, 100, 512, 1024, "swiglu", True), (40, 100, 576, 960, "silu", False),
    (3, 150, 576, 640, "swiglu", True), (2, 90, 512, 512, "relu", False)])
def test_accumulated_weight_gradients(E, rows, d, f, act, h_on_load):
    """MOE_ACCUMULATE_DW adds the very gradient that the plain call writes: one
    float32 addition per element."""
    T, k = E * rows, 1
    rng = np.random.Generator(np.random.PCG64(E + d))
    ids = rng.permutation(np.repeat(np.arange(E), rows)).astype(np.int32)[:, None]
    x, dy = _bf16(rng, (T, d), 1.0), _bf16(rng, (T, d), 1.0)
    w1, w3, w2 = (_bf16(rng, (E, d, f), d ** -0.5), _bf16(rng, (E, d, f), d ** -0.5),
                  _bf16(rng, (E, f, d), f ** -0.5))
    gates = torch.from_numpy(rng.random((T, 1), dtype=np.float32)).cuda()
    A0, B0 = _bf16(rng, (T, f), 1.0), _bf16(rng, (T, f), 1.0)
    ix = oracle.build_index(ids, E)
    off, eti, ss = dev(ix.offsets), dev(ix.eti), dev(ix.slot_src)
    gated = act == "swiglu"
    base = [torch.randn(s, device="cuda") for s in ((E, d, f), (E, d, f), (E, f, d))]

    def run(flags, dw):
        fl = flags | B.ACT_FLAG[act] | (B.MOE_H_ON_LOAD if h_on_load else 0)
        n = B.moe_ffn_bwd_workspace_size(T, d, f, E, k, fl)
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
        dg = torch.empty((T, 1), dtype=torch.float32, device="cuda")
        dX = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        B.moe_ffn_bwd(dy, x, w1, w3 if gated else None, w2, gates, off, eti, ss, A0.clone(),
                      B0.clone() if gated else None, T, d, f, E, k, fl, dw[0],
                      dw[1] if gated else None, dw[2], dg, dX, ws, n)
        torch.cuda.synchronize()
        return dw

    plain = run(0, [torch.full_like(b, float("nan")) for b in base])
    acc = run(B.MOE_ACCUMULATE_DW, [b.clone() for b in base])
    for i in (0, 1, 2) if gated else (0, 2):
        assert torch.equal(acc[i], base[i] + plain[i]), i

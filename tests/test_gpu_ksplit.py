"""The matrix-core GEMM of more than 32 tokens: each tile size with the
reduction split over a workgroup's waves and the many-token kernels, with
remainders in tokens, columns and channels and several tiles a workgroup,
against the sum in fp64.

Bound: y is a sum of d_in products, each exact in fp32, in some order, times
two scales: d_in + 2 roundings of relative size 2^-24 on partial sums no larger
than sum |a_p w_p|; twice that is allowed."""
import numpy as np
import pytest

from oracle import oasis_oracle as O
from paper_2507_23035_amd import oasis, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# tests/test_routes_cpu.py holds every case to the kernel it is listed under
KS32, KS64, KS128x64, KS128, TILES, PREFILL = 1, 2, 3, 4, 5, 6
CASES = [
    # n, d_in, d_out, seed, kernel         tile (columns x tokens)
    (33, 512, 100, 1, KS32),         # 32 x 32: a token in the second tile, 4 blocks for 16 waves
    (64, 4096, 520, 2, KS32),        # whole token tiles
    (40, 72, 37, 3, KS32),           # a masked last block, d_out not a multiple of 4
    (2047, 64, 70, 10, KS32),        # one block: all waves but one have none
    (36, 4096, 4388, 19, KS32),      # 276 tiles: a second one for some workgroups
    (35, 1032, 4261, 20, KS32),      # the same, masked, unaligned rows of y
    (36, 512, 4302, 21, KS64),       # 64 x 64
    (100, 2056, 8002, 5, KS64),      # a masked last block, unaligned rows of y
    (344, 512, 5432, 11, KS64),      # 510 tiles
    (195, 520, 8308, 12, KS64),      # 520 tiles, masked
    (130, 1024, 8000, 4, KS128x64),  # 128 x 64: two tokens in the last token tile
    (250, 1024, 8070, 6, KS128x64),  # 64 x 4 tiles
    (230, 1208, 8003, 7, KS128x64),  # masked, 18.9 blocks over 8 waves
    (391, 512, 8215, 13, KS128x64),  # 455 tiles
    (328, 520, 8222, 14, KS128x64),  # 390 tiles, masked
    (500, 2048, 8070, 8, KS128),     # 128 x 128
    (641, 512, 8949, 15, KS128),     # 420 tiles
    (1100, 512, 7268, 18, TILES),    # 256 x 128: 9 token tiles, numbered in groups of 8 and 1
    (1000, 1544, 8100, 9, PREFILL),  # 128 x 128 masked: two workgroups on every CU
    (321, 520, 8212, 16, PREFILL),   # one token in the last token tile
    (2135, 520, 2080, 17, PREFILL),  # 17 token tiles
]


@pytest.mark.parametrize("n,d_in,d_out,seed,kernel", CASES)
@pytest.mark.parametrize("accumulate", [False, True])
def test_ksplit_gemm(n, d_in, d_out, seed, kernel, accumulate):
    L = synth.make_layer(synth.custom(n, d_in, d_out, 1, seed=seed))
    print(f"case ksplit n={n} d_in={d_in} d_out={d_out} accumulate={accumulate}", flush=True)
    assert oasis.load().oasis_gemm_route(n, d_in, d_out) == kernel
    dev = torch.device("cuda:0")
    idx_w = torch.from_numpy(oasis.pack_weight_indices(L.w_idx).view(np.int32)).to(dev)
    s_w = torch.from_numpy(L.s_w).to(dev)
    lut = oasis.build_lut(L.cb_a, 4, L.cb_w, 4)
    q = O.quantize_act(L.x, L.cb_a, 4, 0)
    idx_act = torch.from_numpy(O.pack_act_indices(q["a"])).to(dev)
    t = torch.from_numpy(q["t"]).to(dev)
    # y at a 16-byte address, then 4 bytes past one (stored by elements)
    ys = []
    for off in (0, 1):
        y = torch.full((n * d_out + off,), 0.5 if accumulate else float("nan"), device=dev)
        y = y[off:].view(n, d_out)
        oasis.lut_gemm(idx_act, t, idx_w, s_w, lut, 4, 4, y=y, accumulate=accumulate)
        ys.append(y)
    torch.cuda.synchronize()
    a = torch.from_numpy(L.cb_a.astype(np.float64)[q["a"]] * q["t"].astype(np.float64)[:, None])
    w = torch.from_numpy(L.cb_w.astype(np.float64)[L.w_idx] * L.s_w.astype(np.float64)[None, :])
    ref = a @ w
    bound = 2.0 * (d_in + 2) * 2.0 ** -24 * (a.abs() @ w.abs())
    if accumulate:  # 0.5 added once, one more rounding
        ref = ref + 0.5
        bound = bound + 2.0 ** -23 * (ref.abs() + 0.5)
    for y in ys:
        err = (y.cpu().double() - ref).abs()
        assert bool((err <= bound).all()), float((err / bound).max())

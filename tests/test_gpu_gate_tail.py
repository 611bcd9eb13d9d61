"""GPU parity of the row lengths of the post-EC tail's RMSNorm and of the token
counts and widths of the tanh-MLP gate, against the float64 oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import spear_oracle as O
from paper_2606_11244_amd import synth as S

from gpu_util import assert_parity, gpu_y, log, scaled_ec, zero_weight

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N", [8, 20, 2040, 2048, 2056, 4096, 4104, 8192, 8200, 16392, 32768, 32776])
@pytest.mark.parametrize("dt", [S.F16, S.BF16])
def test_rmsnorm_row_lengths(N, dt):
    """Rows of whole 16-byte chunks at every chunk count per thread and its
    edges, and rows past them (20: not whole chunks; 32776: too long). The
    norm's own error is one rounding of its inputs' fp32 function, far inside
    the bar."""
    from paper_2606_11244_amd import spear as sp
    L = S.make_layer(M=3, N=N, K=128, group_size=128, rank=0, act_dtype=dt, seed=N)
    t = S.make_tail(L, seed=1)
    tdt = sp._TORCH_DT[dt]
    res = torch.from_numpy(t["residual"].view(np.int16)).view(tdt).cuda()
    nw = torch.from_numpy(t["norm_w"].view(np.int16)).view(tdt).cuda()
    dl = sp.DeviceLayer(L)
    prob = dl.problem()
    yn = torch.full((3, N), 7.0, dtype=tdt, device="cuda")
    log(f"rmsnorm N={N} dt={dt}")
    dl.run_tail(prob, sp.allocate_workspace(prob, False), residual=res, norm_w=nw, eps=t["eps"],
                y_norm=yn, with_ec=False)
    torch.cuda.synchronize()
    y = dl.y.float().cpu().numpy().astype(np.float64)
    w = S.from_bits(t["norm_w"], dt).astype(np.float64)
    ref = y / np.sqrt((y * y).mean(axis=1, keepdims=True) + t["eps"]) * w
    # one rounding to the activation dtype of an fp32 result: half an ulp plus
    # fp32 noise of the sum (2^-24 per term, relative, on the scale)
    ulp = 2.0 ** (-11 if dt == S.F16 else -8)
    got = yn.float().cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1.01 * ulp * np.abs(ref) + 1e-7), np.abs(got - ref).max()


# (M, rank, hidden, path): token groups of four and their remainders, ranks and
# hidden widths with and without whole 16-byte parameter rows, the largest
# hidden width (four tokens at once), one producer and several
TANH = [(1, 8, 0, 4), (5, 12, 20, 4), (16, 32, 128, 4), (17, 33, 40, 4), (40, 64, 256, 4),
        (3, 16, 1024, 4), (130, 20, 72, 4), (1, 32, 128, 1), (9, 64, 256, 1), (4, 24, 1000, 1),
        (6, 16, 64, 5), (31, 12, 30, 5), (2, 5, 17, 5), (50, 16, 64, 2), (140, 9, 33, 2), (7, 32, 96, 3)]


@pytest.mark.parametrize("M,rank,h,path", TANH)
@pytest.mark.parametrize("dt", [S.F16, S.BF16])
def test_tanh_gate_shapes(M, rank, h, path, dt):
    """The EC term alone (zero weight, EC x 30), so that the bar applies to the
    gate and not to the product that hides it."""
    L = S.make_layer(M=M, N=80, K=512, group_size=128, rank=rank, act_dtype=dt,
                     gate_kind=S.GATE_TANH_MLP, gate_hidden=h, seed=M * 7 + rank)
    L = scaled_ec(zero_weight(L), 30)
    log(f"tanh M={M} r={rank} h={h} path={path} dt={dt}")
    assert_parity(gpu_y(L, path=path), O.w4ec_linear(L), f"tanh path={path}")


# (roles, M, N, K, slices): every GEMM's epilogue, whole and ragged tiles; the
# 256 x 256 tiles store a call without a residual otherwise than one with it
RES = [(1, 70, 200, 1024, 2), (1, 300, 136, 1024, 1), (2, 300, 200, 1024, 1), (2, 256, 128, 512, 1), (3, 512, 256, 512, 1),
       (3, 257, 300, 1024, 1), (3, 300, 1000, 1024, 1), (4, 20, 200, 1024, 1), (4, 64, 130, 1024, 2), (4, 96, 256, 2048, 4),
       (4, 300, 136, 1024, 1)]


@pytest.mark.parametrize("roles,M,N,K,slices", RES)
@pytest.mark.parametrize("rank", [0, 20])
@pytest.mark.parametrize("dt", [S.F16, S.BF16])
def test_residual_epilogues(roles, M, N, K, slices, rank, dt):
    """A residual of zeros changes no value, a random one meets the oracle,
    and nothing is written past the last row."""
    from paper_2606_11244_amd import spear as sp
    L = S.make_layer(M=M, N=N, K=K, group_size=128, rank=rank, act_dtype=dt, seed=M + N, ec_std=0.05)
    res = S.make_tail(L, seed=2)["residual"]
    tdt = sp._TORCH_DT[dt]
    dl = sp.DeviceLayer(L)
    prob = dl.problem(force_path=4)
    y = torch.full((M + 4, N), 7.0, dtype=tdt, device="cuda")

    def call(r):
        y.fill_(7.0)
        if r is None:
            (dl.run_ec if rank else dl.run_w4)(prob, ws, y=y[:M])
        else:
            dl.run_tail(prob, ws, residual=r, y=y[:M], with_ec=rank > 0)
        torch.cuda.synchronize()
        assert torch.all(y[M:] == 7.0)
        return y[:M].clone()

    sp.set_gemm_tile(256 if roles in (2, 3) else 0)
    sp.set_gemm_slices(slices)
    sp.set_gemm_roles(roles)
    try:
        log(f"residual roles={roles} M={M} N={N} K={K} S={slices} r={rank} dt={dt}")
        ws = sp.allocate_workspace(prob, rank > 0)
        plain = call(None)
        assert torch.equal(plain, call(torch.zeros_like(plain)))
        got = call(torch.from_numpy(res.view(np.int16)).view(tdt).cuda())
    finally:
        sp.set_gemm_roles(0)
        sp.set_gemm_slices(0)
        sp.set_gemm_tile(0)
    ref = O.w4ec_linear(L) if rank else O.w4_linear_layer(L)
    assert_parity(plain.double().cpu().numpy(), ref, "plain")
    assert_parity(got.double().cpu().numpy(), ref + S.from_bits(res, dt).astype(np.float64), "residual")

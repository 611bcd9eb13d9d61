"""GPU parity of the GEMM that keeps the codes in registers (17 to 384 tokens):
its token-tile widths, K-slices and remainders, ragged rows, both code widths,
the EC epilogue, and grouped calls that share its launch and the EC
pre-kernel's, bit for bit the members' own calls."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import spear_oracle as O
from paper_2606_11244_amd import synth as S

from gpu_util import assert_parity, gpu_y, log, scaled_ec, with_fields, zero_weight

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


@pytest.fixture
def forced():
    """The kernel for every GEMM call above 16 tokens, in `slices` K-slices."""
    from paper_2606_11244_amd import spear as sp

    def set_(slices=0):
        sp.set_gemm_roles(4)
        sp.set_gemm_slices(slices)
    yield set_
    sp.set_gemm_roles(0)
    sp.set_gemm_slices(0)


# (M, N, K, G, slices): every token-tile width and its edges, two and three
# token tiles, iteration counts around the stages in flight (1, 5, 6, 7, 13
# iterations per slice), rows past a tile, one group and many per slice
SHAPES = [(17, 128, 128, 128, 1), (32, 130, 640, 0, 1), (33, 100, 768, 128, 1), (48, 256, 896, 128, 1),
          (49, 40, 1664, 128, 2), (64, 384, 2048, 256, 4), (65, 129, 1536, 128, 2), (96, 300, 3328, 0, 2),
          (97, 16, 1024, 128, 8), (128, 128, 2048, 1024, 4), (129, 200, 1152, 128, 1), (200, 64, 2304, 0, 2),
          (300, 1040, 1024, 128, 2), (40, 2, 6656, 128, 4)]


@pytest.mark.parametrize("M,N,K,G,slices", SHAPES)
@pytest.mark.parametrize("dt,bits", [(S.F16, 4), (S.BF16, 4), (S.F16, 3), (S.BF16, 3)])
def test_product(forced, M, N, K, G, slices, dt, bits):
    L = S.make_layer(M=M, N=N, K=K, group_size=G, rank=0, act_dtype=dt, seed=M + N, weight_bits=bits)
    forced(slices)
    log(f"mid M={M} N={N} K={K} G={G} S={slices} dt={dt} bits={bits}")
    assert_parity(gpu_y(L, path=4, with_ec=False), O.w4_linear_layer(L), "product")


@pytest.mark.parametrize("M,slices", [(20, 1), (40, 2), (64, 1), (90, 1)])
@pytest.mark.parametrize("dt,bits", [(S.F16, 4), (S.BF16, 4), (S.BF16, 3)])
def test_infinite_nan_and_huge_activations(forced, M, slices, dt, bits):
    """Infinities, NaN and (bf16) values whose products with the biased codes
    would overflow: what the other GEMM (k_gemm) gives, infinities with their
    signs, NaN where a zero weight meets an infinity, and the oracle's values
    in the tokens that stay finite."""
    from paper_2606_11244_amd import spear as sp
    L = S.make_layer(M=M, N=200, K=1024, group_size=128, rank=0, act_dtype=dt, seed=M, weight_bits=bits)
    x = S.from_bits(L.x, dt).copy()
    x[3, 77], x[7, 11], x[9, 1000] = np.inf, -np.inf, np.nan
    if dt == S.BF16:
        x[5, 300], x[M - 1, 640] = 3e37, -2.5e38
    L = with_fields(L, x=S.to_bits(x, dt))
    sp.set_gemm_roles(1)
    ref = gpu_y(L, path=4, with_ec=False)
    forced(slices)
    log(f"mid nonfinite M={M} S={slices} dt={dt} bits={bits}")
    got = gpu_y(L, path=4, with_ec=False)
    assert np.isinf(ref[[3, 7]]).mean() > 0.5 and np.isnan(ref[9]).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
    rows = [m for m in range(M) if m not in (3, 7, 9)]
    want = O.w4_linear_layer(L)[rows]
    assert np.isfinite(got[rows]).all()
    # per token: the huge ones must not hide the others
    for m, y in zip(rows, want):
        assert_parity(got[m:m + 1], y[None], f"token {m}")


@pytest.mark.parametrize("M,N,K,rank,slices,int8", [
    (20, 200, 1024, 16, 1, False), (33, 130, 1024, 7, 2, True), (64, 256, 2048, 64, 4, True),
    (96, 100, 1024, 33, 1, False), (128, 128, 1024, 256, 1, False), (70, 90, 1024, 200, 8, True),
    (130, 140, 2048, 24, 2, False)])
@pytest.mark.parametrize("dt", [S.F16, S.BF16])
def test_ec_epilogue(forced, M, N, K, rank, slices, int8, dt):
    """The EC term alone, so that the bar applies to it, and the whole layer."""
    L = S.make_layer(M=M, N=N, K=K, group_size=128, rank=rank, act_dtype=dt, seed=M + rank, ab_int8=int8)
    forced(slices)
    log(f"mid EC M={M} N={N} r={rank} S={slices} int8={int8} dt={dt}")
    assert_parity(gpu_y(L, path=4), O.w4ec_linear(L), "layer")
    Z = zero_weight(L) if int8 else scaled_ec(zero_weight(L), 30)
    assert_parity(gpu_y(Z, path=4), O.w4ec_linear(Z), "EC term")


def _group_check(M, K, ranks, Ns=(520, 128, 1100), launches=None, **kw):
    """A group's outputs are the members' own calls' (bit for bit, on one
    workspace twice in a row) and meet the oracle."""
    from paper_2606_11244_amd import spear as sp
    dls, members, alone = [], [], []
    for i, (N, r) in enumerate(zip(Ns, ranks)):
        dl = sp.DeviceLayer(S.make_layer(M=M, N=N, K=K, rank=r, seed=M + i, ec_std=0.05, **dict(dict(group_size=128), **kw)))
        prob = dl.problem()
        ws = sp.allocate_workspace(prob, r > 0)
        y = torch.empty_like(dl.y)
        (dl.run_ec if r > 0 else dl.run_w4)(prob, ws, y=y)
        dls.append(dl)
        alone.append(y)
        members.append(dl.member(prob, with_ec=r > 0))
    log(f"group M={M} K={K} ranks={ranks} Ns={Ns} {kw} launches={sp.group_launches(members)}")
    assert launches is None or sp.group_launches(members) == launches
    ws = torch.zeros(max(256, sp.group_workspace(members)), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        for dl in dls:
            dl.y.fill_(7.0)
        sp.w4ec_linear_group(members, ws)
        torch.cuda.synchronize()
        for dl, y in zip(dls, alone):
            assert torch.equal(dl.y.view(torch.int16), y.view(torch.int16))
    for dl, r in zip(dls, ranks):
        got = dl.y.float().cpu().numpy().astype(np.float64)
        assert_parity(got, O.w4ec_linear(dl.layer) if r else O.w4_linear_layer(dl.layer), "group")


# (M, K, ranks, launches): the counts test_group.py derives on the host
@pytest.mark.parametrize("M,K,ranks,launches", [
    (24, 1024, (0, 0, 0), 1), (20, 1024, (32, 32, 32), 2), (24, 8192, (16, 0, 16), 2), (40, 2048, (64, 0, 64), 2),
    (64, 1024, (24, 33, 0), 2), (90, 2048, (0, 32, 0), 2), (300, 1024, (32, 64, 32), 4), (8, 4096, (32, 32, 0), 3),
    (20, 1024, (0, 32, 0), 2),
    (1, 8192, (64, 64, 64), 2), (4, 8192, (64, 0, 64), 3), (16, 8192, (64, 20, 64), 2), (32, 8192, (32, 64, 32), 2)])
def test_group_is_the_members_own_calls(M, K, ranks, launches):
    """Products that share a launch, EC pre-kernels that share one (also where
    the products do not: at 300 tokens of a small layer), and producer-fused
    decode calls whose projections move to the shared pre-kernel, alone and
    beside members that share nothing."""
    _group_check(M, K, ranks, launches=launches)


@pytest.mark.parametrize("kw", [
    dict(act_dtype=S.BF16), dict(act_dtype=S.BF16, weight_bits=3, group_size=0), dict(weight_bits=3),
    dict(act_dtype=S.BF16, ab_int8=True), dict(ab_int8=True, gate_kind=S.GATE_ONE),
    dict(gate_kind=S.GATE_TANH_MLP, gate_hidden=72), dict(act_dtype=S.BF16, gate_kind=S.GATE_TANH_MLP, gate_hidden=128),
    dict(act_dtype=S.BF16, gate_kind=S.GATE_ONE, weight_bits=3)])
@pytest.mark.parametrize("M,K,ranks", [(8, 4096, (32, 24, 32)), (3, 8192, (64, 20, 64)), (20, 1024, (32, 0, 24)),
                                       (40, 2048, (64, 33, 64))])
def test_group_kinds(M, K, ranks, kw):
    """The shared pre-kernel with the shared GEMV (8 tokens; 3 tokens, members
    that are producer-fused alone) and with the shared k_gemm_r, over the
    dtypes, code widths, factor formats and gates."""
    _group_check(M, K, ranks, launches=2, **kw)


@pytest.mark.parametrize("M", [4, 16])
@pytest.mark.parametrize("kw", [dict(), dict(act_dtype=S.BF16, ab_int8=True)])
def test_group_four_row_tiles(M, kw):
    """Producer-fused members of four row tiles (more than 8192 rows, K 8192)
    beside narrower ones, which are brought to four in the shared launch."""
    from paper_2606_11244_amd import spear as sp
    plans = [sp.dispatch_plan(sp.problem(M, N, 8192, 128, sp.F16, 64)) for N in (8224, 1100)]
    assert [(p.path, p.tile_n) for p in plans] == [(sp.PATH_FUSED_GEMV, 64), (sp.PATH_FUSED_GEMV, 32)]
    _group_check(M, 8192, (64, 64), Ns=(8224, 1100), launches=2, **kw)


@pytest.mark.parametrize("M,N,K,rank", [
    (33, 4100, 2048, 16), (64, 4100, 2048, 8), (96, 4200, 8192, 16), (129, 300, 1024, 24), (192, 8200, 1024, 12),
    (193, 260, 2944, 24), (300, 260, 2944, 16), (384, 130, 2944, 0)])
@pytest.mark.parametrize("dt,bits", [(S.F16, 4), (S.BF16, 4), (S.BF16, 3)])
def test_auto_takes_it(M, N, K, rank, dt, bits):
    """AUTO at the edges of its sizes: the plan is the one that forcing the
    kernel gives, and not the one of the other kernels, and whole layers meet
    the oracle."""
    from paper_2606_11244_amd import spear as sp
    L = S.make_layer(M=M, N=N, K=K, group_size=128, rank=rank, act_dtype=dt, seed=M + N, weight_bits=bits)

    def plan(roles):
        sp.set_gemm_roles(roles)
        try:
            return sp.dispatch_plan(sp.problem(M, N, K, 128, dt, rank, L.gate_kind, 0, sp.PATH_AUTO, bits),
                                    rank > 0).as_dict()
        finally:
            sp.set_gemm_roles(0)
    assert plan(0) == plan(4) != plan(1)
    log(f"mid AUTO M={M} N={N} K={K} r={rank} dt={dt} bits={bits}")
    ref = O.w4ec_linear(L) if rank else O.w4_linear_layer(L)
    assert_parity(gpu_y(L, path=0, with_ec=rank > 0), ref, "auto")

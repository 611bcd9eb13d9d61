"""GPU parity of the decode GEMV over its K-slices: one slice (the build without
the reduction), and counts below, at and past the four that are summed
together, on every variant; and groups whose members differ in slices."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import spear_oracle as O
from paper_2606_11244_amd import synth as S

from gpu_util import assert_parity, gpu_y, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


@pytest.mark.parametrize("slices", [1, 2, 4, 5, 6, 9])
@pytest.mark.parametrize("M,rank,gate,int8", [
    (1, 16, S.GATE_SIGMOID_LINEAR, False), (5, 12, S.GATE_TANH_MLP, False), (16, 16, S.GATE_ONE, True),
    (3, 40, S.GATE_SIGMOID_LINEAR, False), (16, 32, S.GATE_TANH_MLP, False)])
@pytest.mark.parametrize("dt,bits", [(S.F16, 4), (S.BF16, 4), (S.BF16, 3)])
def test_slices(slices, M, rank, gate, int8, dt, bits):
    """The product alone and the producer-fused, semi-fused and local variants
    in `slices` K-slices, twice on one workspace."""
    from paper_2606_11244_amd import spear as sp
    L = S.make_layer(M=M, N=90, K=2304, group_size=128, rank=rank, act_dtype=dt, seed=M + rank, ec_std=0.05,
                     gate_kind=gate, gate_hidden=24 if gate == S.GATE_TANH_MLP else 0, ab_int8=int8, weight_bits=bits)
    ref, ref4 = O.w4ec_linear(L), O.w4_linear_layer(L)
    paths = [1, 4] + ([5] if rank <= 16 else [])
    sp.set_gemv_shape(k_slices=slices)
    try:
        for path in [0] + paths:
            dl = sp.DeviceLayer(L)
            ec = path > 0
            prob = dl.problem(force_path=path if ec else 1)
            assert sp.dispatch_plan(prob, ec).split_k == slices
            ws = sp.allocate_workspace(prob, ec)
            log(f"slices S={slices} M={M} r={rank} path={path} dt={dt} bits={bits}")
            y = gpu_y(L, prob.force_path, with_ec=ec, workspace=ws, dev=dl)
            assert_parity(y, ref if ec else ref4, f"path={path}")
            assert np.array_equal(y, gpu_y(L, prob.force_path, with_ec=ec, workspace=ws, dev=dl))
    finally:
        sp.set_gemv_shape()


@pytest.mark.parametrize("M,Ks,rank", [(1, (512, 4096, 2048), 16), (8, (1024, 4096), 8), (2, (1024, 8192), 0),
                                       (4, (512, 4096), 40)])
def test_group_of_different_slices(M, Ks, rank):
    """Members of one slice beside members of several in one launch."""
    from paper_2606_11244_amd import spear as sp
    dls, members, alone, splits = [], [], [], []
    for i, K in enumerate(Ks):
        dl = sp.DeviceLayer(S.make_layer(M=M, N=256, K=K, group_size=128, rank=rank, seed=K, ec_std=0.05))
        prob = dl.problem()
        y = torch.empty_like(dl.y)
        (dl.run_ec if rank else dl.run_w4)(prob, sp.allocate_workspace(prob, rank > 0), y=y)
        splits.append(sp.dispatch_plan(prob, rank > 0).split_k)
        dls.append(dl)
        alone.append(y)
        members.append(dl.member(prob, with_ec=rank > 0))
    log(f"group slices M={M} Ks={Ks} r={rank} splits={splits} launches={sp.group_launches(members)}")
    assert len(set(splits)) > 1
    ws = torch.zeros(sp.group_workspace(members), dtype=torch.uint8, device="cuda")
    sp.w4ec_linear_group(members, ws)
    torch.cuda.synchronize()
    for dl, y in zip(dls, alone):
        assert torch.equal(dl.y.view(torch.int16), y.view(torch.int16))

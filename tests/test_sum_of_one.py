"""Contracting Dots of which only one member has any K (experts' weight gradients whose filled capacity slots all lie in the first shard): nothing is
summed, so the launch takes the kernel that the estimate was made for, and gives the bits that the members' joined sum gives."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
import workloads as wl
from tests.harness import Staged
from tests.pin import BY_RULE, MFMA, MID, PAIR, last, pinned


def _wgrad(E, C, M, H, P):
    """Experts' weight gradient, the capacity slots split over P members."""
    return wl.DotWorkload(name="moe_wgrad", cfg=13, dtype="bf16", out_dtype="bf16", lhs_shape=(E, C, M), rhs_shape=(E, C, H), lhs_batch=(0,), rhs_batch=(0,),
                          lhs_contract=(1,), rhs_contract=(1,), mesh_shape=(P,), device_ids=tuple(range(P)), lhs_map=(-1, 0, -1), rhs_map=(-1, 0, -1),
                          out_map=(-1, -1, -1), rhs_sigma=1.0, einsum="ECM,ECH->EMH")


def _taken(E, C, M, H, P, fill):
    """What a grouped call would run (nothing is launched, addresses are not used)."""
    w = _wgrad(E, C, M, H, P)
    mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((0,), (0,), (1,), (1,))
    sh = [g.Sharding(s, m if P > 1 else (-1, -1, -1)) for s, m in ((w.lhs_shape, w.lhs_map), (w.rhs_shape, w.rhs_map), (w.out_shape, w.out_map))]
    bufs = [[g.ShardBuf((1 << 40) + (t * P + (p if t < 2 else 0) << 34), g.BF16) for p in range(P)] for t in range(3)]
    g.grouped_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], fill, 1 << 45, g.dot_workspace_bytes(mesh, dims, *sh, -1, True))
    return last()


@pytest.mark.parametrize("E,C,M,H,filled", [(4, 1024, 4096, 8192, 256), (4, 1024, 4096, 8192, 300), (2, 512, 2048, 1024, 200), (8, 2048, 512, 512, 1024)])
def test_the_kernel_that_was_priced_runs(E, C, M, H, filled):
    with pinned(dry_run=True):
        alone = _taken(E, C, M, H, 1, [filled] * E)
        assert _taken(E, C, M, H, 2, [filled] * E) == (alone[0], 0, 1)
    for kernel in (MFMA, MID, PAIR):
        with pinned(kernel, dry_run=True):
            assert _taken(E, C, M, H, 2, [filled] * E)[0] == kernel
    with pinned(MID, dry_run=True):                  # one expert's slots reach into the second shard: a sum again
        assert _taken(E, C, M, H, 2, [filled] * (E - 1) + [C]) == (MID, 0, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", [BY_RULE, MFMA, MID, PAIR])
def test_same_bits(kernel):
    E, C, M, H, fill = 3, 160, 264, 392, [64, 80, 7]
    w = _wgrad(E, C, M, H, 2)
    lhs, rhs = wl.draw_normal_bf16(1, w.lhs_shape), wl.draw_normal_bf16(2, w.rhs_shape)
    raw = []
    for fills, k, one_launch in ((fill, kernel, BY_RULE), (fill, MFMA, 0)):
        st = Staged(w, lhs, rhs)
        with pinned(k, 0, one_launch):
            st.run_grouped(fill=fills)
            assert k == BY_RULE or last()[0] == k
        raw.append(st.out[0][1].view(torch.int16).cpu())
    assert torch.equal(*raw)
    ref = np.stack([wl.bf16_bits_to_f64(lhs[e, :f]).T @ wl.bf16_bits_to_f64(rhs[e, :f]) for e, f in enumerate(fill)])
    got = st.out_shard(0)
    assert np.linalg.norm(got - ref) <= 4e-3 * np.linalg.norm(ref)          # one rounding to bf16: 2^-9 relative at most

"""GPU parity of SAME replica growth (Sec. 3 annealing) through the C ABI:
bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1511_06416_amd as same
from tests import gpu_helpers as H
from workloads import Network, make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    same.load_library()


@pytest.mark.parametrize("cfg,kw,m2", [(4, dict(m=2), 7), (5, dict(n_cols=3_001, m=3), 10), (1, {}, 1)])
def test_grow_replicas_matches_oracle(cfg, kw, m2):
    w = make_workload(cfg, **kw)
    st = w.states[0].numpy()
    ref = oracle.grow_replicas(st, m2)
    ctx = H.context_for(w.net)
    dst = torch.full(same.state_shape(w.net.n, m2, w.ld), 77, dtype=w.states[0].dtype, device="cuda")
    same.same_grow_replicas(ctx, same.pack_states(w.states[0]).cuda(), w.m, dst, m2, w.ld)
    torch.cuda.synchronize()
    assert np.array_equal(same.unpack_states(dst.cpu().numpy(), m2), ref)
    # padding slots of the last destination quad follow the same rule (a valid state)
    full = same.unpack_states(dst.cpu().numpy(), 4 * ((m2 + 3) // 4))
    for r in range(m2, full.shape[1]):
        assert np.array_equal(full[:, r], st[:, r % w.m])
    ctx.close()


def test_grow_replicas_int16_ragged_rows():
    card = np.array([300, 3], dtype=np.int32)
    ctx = H.context_for(Network("custom", [[], [0]], card))
    rng = np.random.default_rng(4)
    st = rng.integers(0, 3, (2, 3, 20)).astype(np.int16)  # 20 columns, m = 3 grown to 5
    ref = oracle.grow_replicas(st, 5)
    dst = torch.zeros(same.state_shape(2, 5, 20), dtype=torch.int16, device="cuda")
    same.same_grow_replicas(ctx, torch.from_numpy(same.pack_states(st)).cuda(), 3, dst, 5, 20)
    torch.cuda.synchronize()
    assert np.array_equal(same.unpack_states(dst.cpu().numpy(), 5), ref)
    ctx.close()


@pytest.mark.parametrize("m,m2", [(2, 7), (3, 10), (5, 5)])
def test_grow_replicas_4bit(m, m2):
    w = make_workload(5, n_cols=2_001, m=m)
    st = w.states[0].numpy()
    ref = oracle.grow_replicas(st, m2)
    ctx = H.context_for(w.net, state_bits=4)
    dst = torch.full(same.state_shape(w.net.n, m2, w.ld, 4), -1, dtype=torch.int16, device="cuda")
    same.same_grow_replicas(ctx, H.to_device(ctx, st), m, dst, m2, w.ld)
    torch.cuda.synchronize()
    assert np.array_equal(H.from_device(ctx, dst, m2), ref)
    ctx.close()


@pytest.mark.parametrize("bits", [4, 8, 16])
@pytest.mark.parametrize("m,m2,ld,shift", [
    (1, 1, 4, 0),        # one quad, fewer columns than a lane's
    (4, 13, 2056, 0),    # whole source quads, a second column chunk, 16-byte rows
    (5, 20, 2052, 0),    # wrapped quads; 4-bit rows that start on 8-byte boundaries
    (3, 11, 516, 8),     # arrays that start on 8-byte boundaries
    (6, 9, 260, 2),      # arrays aligned to a 4-bit quad only
])
def test_grow_replicas_paths(bits, m, m2, ld, shift):
    """The widths a lane takes by alignment, over quads that are copied and
    quads that are assembled from one, two and three source quads."""
    K = {4: 16, 8: 100, 16: 300}[bits]
    shift = max(shift, {4: 2, 8: 4, 16: 8}[bits]) if shift else 0
    ctx = H.context_for(Network("custom", [[], [0]], np.array([K, 3], dtype=np.int32)),
                        state_bits=4 if bits == 4 else 0)
    st = np.random.default_rng(m2).integers(0, 3, (2, m, ld)).astype(np.int16 if bits == 16 else np.int8)
    src = H.to_device(ctx, st)

    def place(t):  # the same tensor at an address `shift` bytes past an aligned one
        raw = torch.empty(t.numel() * t.element_size() + 64, dtype=torch.uint8, device="cuda")
        out = raw[shift:shift + t.numel() * t.element_size()].view(t.dtype).view(t.shape)
        return out.copy_(t)

    src = place(src)
    shape = same.state_shape(2, m2, ld, 4 if bits == 4 else bits)
    dst = place(torch.full(shape, -1, dtype=src.dtype, device="cuda"))
    same.same_grow_replicas(ctx, src, m, dst, m2, ld)
    torch.cuda.synchronize()
    assert np.array_equal(H.from_device(ctx, dst, 4 * ((m2 + 3) // 4))[:, :m2], oracle.grow_replicas(st, m2))
    ctx.close()

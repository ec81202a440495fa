"""Step A of the sequence backward where lists have few rows: as many as its loads side by side and one more, against
the sums in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2211_05239_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def recd():
    from paper_2211_05239_amd import recd as mod
    return mod


@pytest.fixture(scope="module")
def ctx(recd):
    c = recd.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("D", [4, 32, 64, 96, 256, 1024])
@pytest.mark.parametrize("most", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("loose", [False, True])
def test_lists_of_few_rows(ctx, D, most, loose):
    """Up to `most` rows a list, all those below it among them; lengths that end within, at and beyond the positions a block
    takes at once; tight and loose bounds; nothing is written beyond the unique ids."""
    rng = np.random.default_rng(10 * D + most)
    F, rows = 2, 500
    feats = []
    for f in range(F):
        lists = [rng.integers(0, rows, n).tolist() for n in [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 65, 130] * 2]
        which = [i for i in range(len(lists)) for _ in range(1 + i % most)]
        which += [0] * (96 * 2 - len(which))
        feats.append([lists[i] for i in rng.permutation(which)])
    batch = synth.batch_from_lists(feats)
    B, N = batch.B, batch.N
    values, offsets, ik = gu.gpu_build(ctx, batch)
    U_cap, M_cap = (F * B, N) if loose else (ik.U, ik.M)
    gout = rng.standard_normal((N, D)).astype(np.float32)
    grad_emb = torch.full((M_cap, D), float("nan"), device="cuda")
    touched = torch.zeros(M_cap, dtype=torch.int64, device="cuda")
    feat_roff = torch.zeros(F + 1, dtype=torch.int64, device="cuda")
    grad_rows = torch.zeros(M_cap, D, device="cuda")
    u_values, u_offsets = ik.u_values, ik.u_offsets
    ctx.backward_sequence_dedup(F, B, gu.to_dev(gout), offsets, ik.inverse, ik.feat_uoff, u_values, u_offsets, [rows] * F,
                                U_cap, M_cap, grad_emb, touched, feat_roff, grad_rows, want_count=True)
    torch.cuda.synchronize()
    uo, fu, inv = u_offsets.cpu().numpy(), ik.feat_uoff.cpu().numpy(), ik.inverse.cpu().numpy().reshape(F, B)
    ref = np.zeros((ik.M, D))
    size = np.zeros((ik.M, D))
    for l in range(F * B):
        u, a, b = fu[l // B] + inv[l // B, l % B], batch.offsets[l], batch.offsets[l + 1]
        ref[uo[u]:uo[u] + b - a] += gout[a:b]
        size[uo[u]:uo[u] + b - a] += np.abs(gout[a:b])
    got = grad_emb.cpu().numpy()
    # at most `most` additions in 32 bits, each off by half a unit of a partial sum no larger than that of the amounts
    assert (np.abs(got[:ik.M] - ref) <= most * 2.0 ** -24 * size).all()
    assert np.isnan(got[ik.M:]).all()

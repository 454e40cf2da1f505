"""How the feature-map kernels deal out their 32-token tiles must not show in the results: with few tiles
a workgroup applies one map, with more it keeps all of them (the line is at 3072 tiles), waves take tiles
in an order that varies, and lanes past the end of a sequence repeat its last token."""
import pytest
import torch

import paper_2602_12128_amd as hla
from paper_2602_12128_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _handle(F, dphi, d, H, max_tokens):
    op = hla.HLA(head_dim=d, feature_dim=dphi, degree=F, io_dtype=hla.HLA_BF16, max_heads=H, max_tokens=max_tokens, max_seqs=2)
    phi = wl.draw_phi_weights(torch.Generator("cpu").manual_seed(5), d, dphi, 1 + F, torch.bfloat16)
    op.set_phi_weights([{k: v.cuda() for k, v in m.items()} for m in phi])
    return op


@pytest.mark.parametrize("F,dphi,d", [(3, 6, 128), (3, 6, 64), (2, 12, 128), (2, 12, 64)])
def test_features_do_not_depend_on_the_split(F, dphi, d):
    H, top = 12, 8500  # 12 x 266 tiles: all maps in one workgroup
    gen = torch.Generator("cuda").manual_seed(7)
    Q, K, V = (torch.randn(1, H, top, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    op = _handle(F, dphi, d, H, top)
    nfeat = (1 + F) * dphi

    def features(n):
        q, k, v = (t[:, :, :n].contiguous() for t in (Q, K, V))
        op.forward(q, k, v, torch.empty_like(v))
        return op.read_workspace(hla.binding.HLA_WS_FEATURES, H * n * nfeat).reshape(H, n, nfeat)

    ref = features(top)
    for n in (1, 33, 700, 8160, 8161, 8192):  # 8160: the last size with one map per workgroup
        assert torch.equal(torch.as_tensor(features(n)), torch.as_tensor(ref)[:, :n]), n


@pytest.mark.parametrize("F,dphi,d,N", [(3, 6, 128, 33), (2, 12, 128, 31), (3, 6, 64, 65), (2, 12, 64, 1)])
def test_rows_past_a_sequence_stay_untouched(F, dphi, d, N):
    B, H, pad = 2, 3, 31  # the rows a ragged tile would reach
    gen = torch.Generator("cuda").manual_seed(11)
    Q, K, V, dO = (torch.randn(B, H, N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    op = _handle(F, dphi, d, H, B * N)
    bufs = [torch.full((B, H, N + pad, d), 77.0, dtype=torch.bfloat16, device="cuda") for _ in range(4)]
    O, dQ, dK, dV = (x[:, :, :N] for x in bufs)
    op.forward(Q, K, V, O)
    op.backward(Q, K, V, O, dO, dQ, dK, dV)
    for x in bufs:
        assert (x[:, :, N:] == 77.0).all()

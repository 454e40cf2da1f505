"""The fp32 matrix-core kernels of the generic path at the edges of their tiles: token counts around
the 64-token (paper's forms) and 32-token (run-time form) tile and around a run of several tiles, forms
with an odd number of monomials, the largest form, and views whose rows cannot be read 16 bytes at a
time, against the CPU oracle.  The bound is the path's 1e-4 of max|ref| (fp32 sums: 1e-6 measured)."""
import pytest
import torch

import paper_2602_12128_amd as hla
from paper_2602_12128_amd import workloads as wl
from tests import parity_utils as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,dphi,d,H,N,lens", [
    (3, 6, 64, 1, 63, None),
    (3, 6, 128, 3, 65, None),
    (2, 12, 128, 2, 129, None),
    (2, 12, 32, 1, 64, None),
    (3, 6, 32, 5, 8200, None),         # more tiles than partial states: runs of several tiles
    (3, 6, 128, 5, 4100, None),        # the same at eight waves (254 partial states), in the two-factor
    (2, 12, 128, 5, 2501, None),       # form (169) and with run-time monomials, an odd number of them (504)
    (3, 5, 64, 5, 3301, None),         # or five row blocks (101)
    (2, 16, 128, 5, 1001, None),
    (3, 5, 64, 2, 33, None),           # 35 monomials: an odd row count
    (1, 256, 32, 1, 31, None),         # 256 monomials of one factor
    (2, 16, 128, 2, 97, None),         # 136 monomials
    (4, 4, 128, 2, 1, None),
    (3, 6, 128, 2, None, [1, 64, 0, 127, 300]),
    (2, 3, 64, 2, None, [5, 0, 70]),
])
def test_tile_edges(F, dphi, d, H, N, lens):
    cu = None
    if lens is not None:
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        N = cu[-1]
    t = wl.make_feature_inputs(3000 + 7 * N + dphi, 1, H, N, d, F, dphi, torch.float32)
    gpu = pu.run_gpu(t, F, dphi, 1e-6, cu_seqlens=cu, path=hla.HLA_PATH_GENERIC)
    ref = pu.run_oracle(t, F, dphi, 1e-6, cu_seqlens=cu)
    # one-token sequences: dQ, dK are what two cancelling terms leave behind
    scale = None
    if lens is not None and 1 in lens:
        scale = pu.short_sequence_rows(t, ref, cu)
    elif N == 1:
        scale = pu.short_sequence_rows(t, ref, [0, 1])
    pu.assert_parity(gpu, ref, 1e-4, f"f32 tiles F={F} dphi={dphi} d={d} N={N}", row_scale=scale)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_off_sixteen_bytes(dtype):
    B, H, N, d, F, dphi = 1, 2, 150, 64, 3, 6
    t = wl.make_feature_inputs(3100, B, H, N, d, F, dphi, dtype)
    h = pu.make_handle(t, F, dphi, 1e-6, None, None, hla.HLA_PATH_GENERIC)

    def shifted(x):  # the same values in rows of d + 3 elements, one element off the allocation's start
        buf = torch.zeros(x.shape[:3] + (x.shape[3] + 3,), dtype=x.dtype, device="cuda")
        v = buf[..., 1:1 + x.shape[3]]
        v.copy_(x)
        return v

    td = {k: shifted(v) for k, v in t.items()}
    out = {"O": shifted(t["V"]), "dQ": shifted(t["Q"]), "dK": shifted(t["K"]), "dV": shifted(t["V"])}
    h.forward(td["Q"], td["K"], td["V"], out["O"])
    h.backward(td["Q"], td["K"], td["V"], out["O"], td["dO"], out["dQ"], out["dK"], out["dV"])
    torch.cuda.synchronize()
    h.destroy()
    ref = pu.run_oracle(t, F, dphi, 1e-6)
    pu.assert_parity({k: v.contiguous().cpu() for k, v in out.items()}, ref, pu.TOL[dtype], "f32 rows off 16 bytes")


@pytest.mark.parametrize("F,dphi,d,B,H,N", [
    (4, 3, 128, 1, 1, 63),     # four key maps: the most accumulators a workgroup holds
    (1, 16, 32, 2, 2, 65),     # all sixteen feature columns
    (2, 7, 64, 1, 1, 1),       # one token; odd d_phi
    (3, 6, 128, 1, 3, 129),
    (3, 6, 32, 1, 9, 4100),    # more tiles than partials: workgroups of several tiles
    (3, 6, 128, 1, 5, 3301),   # and at eight waves
])
def test_feature_map_tile_edges(F, dphi, d, B, H, N):
    t, phi = wl.make_raw_inputs(3200 + N + d, B, H, N, d, F, dphi, torch.float32)
    gpu = pu.run_gpu(t, F, dphi, 1e-6, phi=phi, path=hla.HLA_PATH_GENERIC, weight_grads=True)
    ref = pu.run_oracle(t, F, dphi, 1e-6, phi=phi, weight_grads=True)
    what = f"f32 maps F={F} dphi={dphi} d={d} N={N}"
    if N == 1:  # every gradient but dV is what two cancelling terms leave behind
        scale = pu.short_sequence_rows(t, ref, [0, 1])
        pu.assert_parity(gpu, ref, 1e-4, what, row_scale=scale)
        return
    pu.assert_parity(gpu, ref, 1e-4, what)
    pu.assert_weight_grad_parity(gpu["wg"], ref["wg"], 1e-4, what)


@pytest.mark.parametrize("d", [32, 128])
def test_gelu_over_its_range(d):
    """Maps with W1 = 1, W2 = the first six hidden units, b2 = 0.25 (GELU is above -0.17): the features are
    GELU(q) + 0.25.  GELU is within 3.9e-7 of the exact one over [-9, 9], the sum adds half an ulp of at most
    9.25 (4.8e-7); beyond, the negative side must be zero and the positive the identity."""
    F, dphi, H, N = 3, 6, 1, 3000
    q = torch.zeros(1, H, N, d)
    q[0, 0, :, :dphi] = torch.linspace(-9, 9, N * dphi).reshape(N, dphi)
    q[0, 0, 0, :dphi] = torch.tensor([-10.0, -30.0, -1e4, 12.0, 1e4, 0.0])
    eye = torch.eye(d, device="cuda")
    phi = {"W1": eye, "b1": torch.zeros(d, device="cuda"), "W2": eye[:, :dphi].contiguous(), "b2": torch.full((dphi,), 0.25, device="cuda")}
    op = hla.HLA(head_dim=d, feature_dim=dphi, degree=F, io_dtype=hla.HLA_F32, max_heads=H, max_tokens=N, max_seqs=1)
    op.set_phi_weights([phi] * (1 + F))
    qd = q.cuda()
    op.forward(qd, qd, qd, torch.empty_like(qd))
    nfeat = (1 + F) * dphi
    got = torch.as_tensor(op.read_workspace(hla.binding.HLA_WS_FEATURES, N * nfeat)).reshape(N, 1 + F, dphi).double()
    x = q[0, 0, :, :dphi].double()
    ref = 0.5 * x * torch.special.erfc(-x / 2 ** 0.5) + 0.25
    for m in range(1 + F):
        err = (got[:, m] - ref).abs()
        assert err[1:].max() < 9e-7, err[1:].max()
        assert (err[0] <= ref[0].abs() * 6e-8).all(), err[0]


def test_runs_follow_the_head_count():
    """One handle, the same tokens, other numbers of heads: the runs of tiles are those of the call's heads."""
    F, dphi, d, N = 3, 6, 32, 8200  # five heads: runs of several tiles; one head: of one
    t = wl.make_feature_inputs(3300, 1, 5, N, d, F, dphi, torch.float32)
    h = pu.make_handle(t, F, dphi, 1e-6, None, None, hla.HLA_PATH_GENERIC)

    def step(op, H):
        x = {k: v[:, :H].contiguous().cuda() for k, v in t.items()}
        out = {"O": x["V"], "dQ": x["Q"], "dK": x["K"], "dV": x["V"]}
        out = {k: torch.empty_like(v) for k, v in out.items()}
        op.forward(x["Q"], x["K"], x["V"], out["O"])
        op.backward(x["Q"], x["K"], x["V"], out["O"], x["dO"], out["dQ"], out["dK"], out["dV"])
        torch.cuda.synchronize()
        return out

    for H in (5, 1, 5, 3):
        fresh = pu.make_handle(t, F, dphi, 1e-6, None, None, hla.HLA_PATH_GENERIC)
        want, got = step(fresh, H), step(h, H)
        fresh.destroy()
        for k in want:
            assert torch.equal(got[k], want[k]), (H, k)
    h.destroy()


@pytest.mark.parametrize("spread", [0.02, 0.2, 1.0, 4.0])
def test_gelu_and_its_slope_are_no_further_off_than_with_erf(spread):
    """The error against 64 bits of GELU and GELU' as the fp32 maps form them, beside that of
    h 0.5 (1 + erf(h / sqrt 2)) and its derivative in fp32 with a correctly rounded erf and exp.  W1 = 1;
    the query map has W2 = -1 and is open where GELU < 0, the first key map W2 = 1, so that features are GELU
    itself and dX / d(feature) is GELU' times one rounding, here and there.  2 % for the sample (72000 values a side)."""
    F, dphi, d, H, N = 3, 6, 32, 4, 6000
    gen = torch.Generator("cpu").manual_seed(3400)
    x = torch.randn(1, H, N, d, generator=gen) * spread
    eye = torch.eye(d)
    col = eye[:, :dphi].contiguous()
    zero, one = torch.zeros(d), torch.ones(dphi)
    maps = [{"W1": eye, "b1": zero, "W2": -col, "b2": 0 * one}, {"W1": eye, "b1": zero, "W2": col, "b2": 0 * one}]
    maps += [{"W1": 0 * eye, "b1": zero, "W2": col, "b2": one}] * 2
    op = hla.HLA(head_dim=d, feature_dim=dphi, degree=F, io_dtype=hla.HLA_F32, max_heads=H, max_tokens=N, max_seqs=1)
    op.set_phi_weights([{k: v.cuda() for k, v in m.items()} for m in maps])
    xd = x.cuda()
    V, dO = (torch.randn(1, H, N, d, generator=gen).cuda() for _ in range(2))
    O, dQ, dK, dV = (torch.empty_like(V) for _ in range(4))
    op.forward(xd, xd, V, O)
    op.backward(xd, xd, V, O, dO, dQ, dK, dV)
    nfeat = (1 + F) * dphi
    feat, dfeat = (torch.as_tensor(op.read_workspace(kind, H * N * nfeat)).reshape(H * N, 1 + F, dphi)
                   for kind in (hla.binding.HLA_WS_FEATURES, hla.binding.HLA_WS_FEATURE_GRADS))
    op.destroy()
    h = x.reshape(H * N, d)[:, :dphi]
    hd = h.double()
    cdf = 0.5 * torch.special.erfc(-hd / 2 ** 0.5)
    value, slope = hd * cdf, cdf + hd * torch.exp(-hd * hd / 2) / (2 * torch.pi) ** 0.5
    erf1 = 1.0 + torch.erf((h * 0.70710678118654752440).double()).float()
    value32 = (h * 0.5) * erf1
    pdf32 = 0.39894228040143267794 * torch.exp((-0.5 * h * h).double()).float()
    slope32 = (0.5 * erf1).double().add(hd * pdf32.double()).float()  # one multiply-add
    for m, dX, sign, side in ((0, dQ, -1.0, h < 0), (1, dK, 1.0, h > 0)):
        got = sign * feat[:, m][side].double()
        err = lambda a: ((a - value[side]).norm() / value[side].norm()).item()
        assert err(got) <= 1.02 * err(value32[side].double()), (m, err(got), err(value32[side].double()))
        du = dfeat[:, m]
        side = side & (du != 0) & (feat[:, m] > 0)
        du = du[side]
        err = lambda dx: ((sign * dx.double() / du.double() - slope[side]).norm() / slope[side].norm()).item()
        got = dX.cpu().reshape(H * N, d)[:, :dphi][side]
        want = sign * du * slope32[side]
        assert err(got) <= 1.02 * err(want), (m, err(got), err(want))


def test_more_rows_than_a_grid_dimension_holds():
    """2^24 (batch row, head) pairs of one token each: a workgroup of 256 threads per row is more than the 2^32
    threads a grid takes in one direction.  The rows are alike, and so are the results."""
    F, dphi, d = 1, 1, 32
    gen = torch.Generator("cpu").manual_seed(3500)
    row = {k: torch.randn(1, 1, 1, d, generator=gen).cuda() for k in ("Q", "K", "V", "dO")}
    phi = wl.draw_phi_weights(torch.Generator("cpu").manual_seed(5), d, dphi, 1 + F, torch.float32)

    def step(B, H):
        op = hla.HLA(head_dim=d, feature_dim=dphi, degree=F, io_dtype=hla.HLA_F32, max_heads=H, max_tokens=B, max_seqs=B)
        op.set_phi_weights([{k: v.cuda() for k, v in m.items()} for m in phi])
        x = {k: v.expand(B, H, 1, d) for k, v in row.items()}
        out = [torch.full((B, H, 1, d), 77.0, device="cuda") for _ in range(4)]
        op.forward(x["Q"], x["K"], x["V"], out[0])
        op.backward(x["Q"], x["K"], x["V"], out[0], x["dO"], *out[1:])
        torch.cuda.synchronize()
        op.destroy()
        return out

    for got, want in zip(step(4096, 4096), step(1, 1)):
        assert bool((got == want).all())

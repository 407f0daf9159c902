"""Every compiled variant of the projections against 64-bit sums, by plans that the test chooses: row tiles, wave
shapes, epilogues, and K ranges of one chunk up to more than two rounds of the rings, with a rest of every length.  The
planners pick a part of these for the models that other tests have; a model of another size takes another part.

Inputs: activations of a normal distribution as hi and lo halves, weights as halves, so that the products are exact in
64 bits and only the fp32 sums differ.  Tolerance: n additions in fp32 in any order err by less than n 2^-24 times the
sum of the magnitudes; n = 2 K products (two planes) and up to 16 sums of the waves.  One fragment of a wrong chunk
(eight products) is off by hundreds of times as much."""
import ctypes as C

import pytest
import torch

import hooks as H

pytestmark = pytest.mark.gpu


def tiles(w):
    """[N][K] half -> operand tiles: [N/16][K/32][k/8 % 4][n % 16][8], rows past the last zero."""
    n, k = w.shape
    pad = torch.zeros(((n + 15) // 16 * 16, k), dtype=w.dtype, device=w.device)
    pad[:n] = w
    return pad.view(-1, 16, k // 32, 4, 8).permute(0, 2, 3, 1, 4).contiguous()


def run_one(pid, R, N, K, splits, mode, seed):
    print("plan %d: %d rows x %d columns, K %d in %d, mode %d" % (pid, R, N, K, splits, mode), flush=True)
    g = torch.Generator(device="cuda").manual_seed(seed)
    dev, ws = "cuda", (R + 79) // 80 * 80
    x = torch.randn((R, K), generator=g, device=dev)
    hi = x.half()
    lo = (x - hi.float()).half()
    X = torch.zeros((2, ws + 80, K + 64), dtype=torch.float16, device=dev)
    X[:, R:ws] = float("nan")                              # rows past the last hold anything; the spare rows are zero
    X[0, :R, :K], X[1, :R, :K] = hi, lo
    w = (0.05 * torch.randn((N, K), generator=g, device=dev)).half()
    if mode == H.ARGMAX:                                   # equal columns all over: ties within and across tiles, waves, groups
        w = w[torch.arange(N, device=dev) % 37].contiguous()
    x64, w64 = hi.double() + lo.double(), w.double()
    want, mag = x64 @ w64.t(), (hi.double().abs() + lo.double().abs()) @ w64.abs().t()
    bound = (2 * K + 16) * 2.0 ** -24 * mag
    wt = tiles(w)
    groups = -(-N // H.cols_per_group(pid))
    out = torch.full((splits, R, N), float("nan"), device=dev) if mode == H.PARTIAL else None
    logits = torch.full((R, N), float("nan"), device=dev) if mode == H.ARGMAX else None
    aval = torch.full((R + 1, groups + 1), -7.0, device=dev)
    aidx = torch.full((R + 1, groups + 1), -7, dtype=torch.int32, device=dev)
    act = torch.full((2, ws + 80, N // 2 + 64), 3.0, dtype=torch.float16, device=dev) if mode == H.SWIGLU else None
    sat = torch.zeros(1, dtype=torch.int64, device=dev)
    torch.cuda.synchronize()
    p = lambda t: C.c_void_p(t.data_ptr() if t is not None else None)  # noqa: E731
    used = C.c_int(-1)
    rc = H.lib().hook_project(p(X), p(wt), p(out), p(act), p(logits), p(aval), p(aidx), p(sat), ws, groups + 1, R, N, K, pid, splits, mode, C.byref(used))
    assert rc == 0, "launch failed with %d" % rc
    assert int(sat) == 0
    if mode == H.PARTIAL:
        got = out.double().sum(0)
        assert bool(((got - want).abs() <= bound).all()), "worst %.3g of the bound" % float(((got - want).abs() / bound).max())
    elif mode == H.ARGMAX:
        assert used.value == groups
        assert bool(((logits.double() - want).abs() <= bound).all()), "worst %.3g of the bound" % float(((logits.double() - want).abs() / bound).max())
        cols = H.cols_per_group(pid)
        for j in range(groups):
            part = logits[:, j * cols:(j + 1) * cols]
            best = part.max(1).values
            first = (part == best[:, None]).float().argmax(1) + j * cols     # the lowest of equal columns
            assert torch.equal(aval[:R, j], best) and torch.equal(aidx[:R, j].long(), first), "group %d" % j
        assert bool((aidx[R] == -7).all()) and bool((aidx[:, groups] == -7).all())
    else:                                                  # tiles alternate: gate and up of features 16 j .. 16 j + 15
        f = lambda t: t.view(R, -1, 2, 16).permute(2, 0, 1, 3).reshape(2, R, N // 2)  # noqa: E731
        (gv, uv), (ge, ue) = f(want), f(bound)
        ref = gv * torch.sigmoid(gv) * uv
        tol = 1.1 * uv.abs() * ge + (gv * torch.sigmoid(gv)).abs() * ue + 1.2 * ge * ue + 2.0 ** -20 * ref.abs() + 2.0 ** -24      # d silu <= 1.1; expf, division, hi + lo
        got = act[:, :R, :N // 2].double().sum(0)
        assert bool(((got - ref).abs() <= tol).all()), "worst %.3g of the bound" % float(((got - ref).abs() / tol).max())
        assert bool((act[:, R:] == 3.0).all()) and bool((act[:, :, N // 2:] == 3.0).all())


@pytest.mark.parametrize("cfg", [0, 1, 2])
@pytest.mark.parametrize("mt", [4, 5, 6, 7, 8])
def test_many_rows(mt, cfg):
    """Two row blocks, the second with seven rows only; one chunk, a ring's depth (two to four) and around, and more than two rounds."""
    cs, kw = H.CONFIGS[cfg]
    R, cols, kc = mt * 16 + 7, cs * 64, kw * 32
    for mode in (H.PARTIAL, H.ARGMAX, H.SWIGLU):
        N = cols + (96 if mode == H.SWIGLU else 53)
        for chunks in (1, 2, 3, 4, 5, 6, 7, 8, 9, 11):
            run_one(H.ROWS + 4 * mt + cfg, R, N, chunks * kc, 1, mode, chunks)
        if mode == H.PARTIAL:
            for splits, chunks in ((2, 5), (3, 3)):
                run_one(H.ROWS + 4 * mt + cfg, R, N, splits * chunks * kc, splits, mode, chunks)


@pytest.mark.parametrize("shape", range(len(H.SHAPES)))
def test_few_rows(shape):
    """One to five row tiles, full and with a single row in the last; chunks of 128, of which a ring of 64-wide chunks holds
    three and a ring of 128-wide ones four."""
    for mode in H.SHAPE_MODES[shape]:
        cols = H.cols_per_group(shape)
        N = cols + (32 if mode == H.SWIGLU else 21)
        for R in (1, 16, 17, 32, 33, 48, 49, 64, 65, 80):
            for chunks in (1, 2, 3, 4, 5, 7, 9):
                run_one(shape, R, N, chunks * 128, 1, mode, chunks)
            if mode == H.PARTIAL:
                for splits, chunks in ((2, 2), (3, 5)):
                    run_one(shape, R, N, splits * chunks * 128, splits, mode, chunks)

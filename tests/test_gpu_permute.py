"""The change between the natural and the colour-blocked order at the edges of its runs: with the identity as operator
the SpMV returns its input exactly, whatever the extents, the type and the vectors' alignment."""
import pytest

pytestmark = pytest.mark.gpu

TYPE = {0: "float64", 1: "float32", 4: "float16", 5: "bfloat16"}


@pytest.fixture(scope="module")
def hp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2507_11512_amd import hpgmx
    return hpgmx


# x extents that are multiples of 8, 4, 2 and 1 points, one run per line and several, odd y and z
@pytest.mark.parametrize("dims", [(8, 3, 5), (16, 5, 2), (40, 7, 6), (12, 5, 3), (20, 4, 9), (6, 5, 4), (2, 2, 2), (37, 6, 5),
                                  (3, 3, 2), (264, 10, 11)])
@pytest.mark.parametrize("dtype", [0, 1, 4, 5])
@pytest.mark.parametrize("shift", [0, 1])
def test_identity(hp, dims, dtype, shift):
    import torch
    coef = [0.0] * 27
    coef[13] = 1.0
    P = hp.Problem(dims, levels=1, coef=coef)
    try:
        n = P.N
        x = torch.randn(n + shift, device="cuda").to(getattr(torch, TYPE[dtype]))[shift:]  # shift: off 16 bytes
        out = torch.float64 if dtype == 0 else torch.float32
        y = torch.full((n + shift,), float("nan"), dtype=out, device="cuda")[shift:]
        hp.spmv(P.h, 0, dtype, x, y)
        assert torch.equal(y, x.to(out))
        if dtype < 2:
            X = torch.stack([x, 2 * x, 3 * x])
            Y = torch.full_like(X, float("nan"))
            hp.spmv_batched(P.h, 0, dtype, X, Y)
            assert torch.equal(Y, X)
    finally:
        P.close()

"""GPU: fp32 fully-connected layers large enough for the product from bf16 thirds, at ragged edges (token blocks, tiles, one
and many slices), against 64 bits; and what the thirds cannot carry -- infinities, NaN, values that round to infinity in bf16,
terms below the normal numbers -- which takes the fp32 instruction instead.  n terms in fp32, rounded once per 16: 2e-7 in the
2-norm covers n = 9001 (0.9 of it is what the fp32 instruction shows at 6304 tokens)."""
import pytest
import torch

import paper_2202_13808_amd as dropit

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def layer(ntok, cin, cout, x_scale=1.0, dy_scale=0.02):
    gen = torch.Generator(device=DEV).manual_seed(ntok)
    x = torch.randn(ntok, cin, generator=gen, device=DEV) * x_scale
    return x, torch.randn(ntok, cout, generator=gen, device=DEV) * dy_scale


def thirds(ntok, cin, cout):
    """Whether the library takes bf16 thirds: 128 x 128 is the tile that pads dW least, and enough of them to fill the chip
    with two blocks of 32 tokens each."""
    up = lambda v, tile: (v + tile - 1) // tile * tile
    least = min(up(cout, 64) * up(cin, 128), up(cout, 64) * up(cin, 64))
    tiles = up(cout, 128) // 128 * (up(cin, 128) // 128)
    return cin % 4 == 0 and cout % 4 == 0 and up(cout, 128) * up(cin, 128) <= least and tiles * max((ntok + 31) // 32 // 2, 1) >= 256


def product(x, dy, gamma):
    assert (x.shape[0], x.shape[1]) in ((417, 1028), (8191, 388)) or thirds(*x.shape, dy.shape[1])
    vals, idx = dropit.compress(x, gamma)
    assert dropit.weight_grad_path(x.shape, x.dtype, vals.numel(), dy.shape[1]) == "fma"
    flat = torch.zeros(x.numel(), dtype=torch.float64, device=DEV)
    flat[idx.long()] = vals.double()
    xr = flat.view(x.shape)
    return dropit.weight_grad(vals, idx, x.shape, dy, dy.shape[1]), dy.double().t() @ xr, xr


@pytest.mark.parametrize("ntok,cin,cout,gamma", [
    (700, 1024, 1024, 0.8),       # whole tiles, a partial token block
    (417, 1028, 1500, 0.9),       # the fp32 instruction: 64-wide tiles pad it less
    (417, 1100, 1500, 0.9),       # ragged in both columns, a single token in the last block
    (64, 3068, 3072, 0.6),        # two token blocks, one slice straight into dW
    (33, 3072, 3060, 0.9),        # ... the second one nearly empty
    (8191, 388, 260, 0.7),        # the fp32 instruction, many slices
    (8191, 452, 332, 0.7),        # ragged in both columns, many slices
    (9001, 196, 76, 0.8),         # ... more than a hundred in two tiles
    (6304, 384, 1536, 0.9),
])
def test_sizes(ntok, cin, cout, gamma):
    assert thirds(ntok, cin, cout) == ((ntok, cin) not in ((417, 1028), (8191, 388)))
    got, want, _ = product(*layer(ntok, cin, cout), gamma)
    err = ((got.double() - want).norm() / want.norm()).item()
    print("thirds", ntok, cin, cout, gamma, "%.2e" % err, flush=True)
    assert err < 2e-7


def test_not_finite():
    """The pattern of infinities and NaN is that of the sums in 64 bits, the rest stays as accurate."""
    x, dy = layer(700, 1024, 1024)
    dy[3, 5] = float("inf")
    dy[400, 900] = float("nan")
    x[699, 1000] = float("-inf")
    x[17, 200] = 3.4e38                            # finite, infinite as bf16
    dy[17, :8] = 1e-3
    got, want, _ = product(x, dy, 0.8)
    want32 = want.to(torch.float32)                # (sums beyond fp32 are infinite in either)
    assert torch.equal(torch.isnan(got), torch.isnan(want32))
    finite = torch.isfinite(want32)
    assert torch.equal(torch.isinf(got), torch.isinf(want32)) and torch.equal(got[~finite & ~torch.isnan(got)], want32[~finite & ~torch.isnan(want32)])
    plain = finite.clone()
    plain[:, 200] = False                          # (the column of the large value: its sums cancel nothing, checked below)
    assert ((got.double() - want)[plain].norm() / want[plain].norm()).item() < 2e-7
    large = finite[:, 200]
    assert ((got.double() - want)[large, 200].abs() <= 1e-6 * want[large, 200].abs()).all()


@pytest.mark.parametrize("x_scale,dy_scale", [(1e-33, 1.0), (1.0, 1e-34), (1e-18, 1e-19), (1e30, 1e-36), (1e18, 1e18)])      # (the last: sums of 1e37, a tenth of the largest fp32)
def test_far_from_one(x_scale, dy_scale):
    got, want, _ = product(*layer(700, 1024, 1024, x_scale, dy_scale), 0.8)
    err = ((got.double() - want).norm() / want.norm()).item()
    print("thirds far", x_scale, dy_scale, "%.2e" % err, flush=True)
    assert err < 4e-7                              # the fp32 instruction's bound at 700 tokens, twice over


def subnormal(rows, columns, seed):
    """Values of a few hundred units of 2^-149, either sign: all three parts of the smaller ones are zero in bf16."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    bits = torch.randint(1, 1000, (rows, columns), generator=gen, device=DEV, dtype=torch.int32)
    sign = torch.randint(0, 2, (rows, columns), generator=gen, device=DEV, dtype=torch.int32)
    return (bits | (sign << 31)).view(torch.float32)


@pytest.mark.parametrize("where", ["x", "dy", "all of x"])
def test_sums_of_lost_terms(where):
    """A column of subnormal values against values of 1e30: its sums are ordinary numbers, and all that the thirds carry of
    them can be exactly zero."""
    x, dy = layer(700, 1024, 1024, 1.0 if where != "dy" else 1e30, 1.0 if where == "dy" else 1e30)
    if where == "x":
        x[:, 200:210] = subnormal(700, 10, 1)
    elif where == "dy":
        dy[:, 900:910] = subnormal(700, 10, 2)
    else:
        x = subnormal(700, 1024, 3)
    got, want, _ = product(x, dy, 0.0)
    part = (slice(900, 910), slice(None)) if where == "dy" else (slice(None), slice(200, 210))
    err = ((got.double() - want)[part].norm() / want[part].norm()).item()
    print("thirds lost", where, "%.2e" % err, "largest", want[part].abs().max().item(), flush=True)
    assert err < 4e-7
    assert ((got.double() - want).norm() / want.norm()).item() < 4e-7


def test_leading_parts_that_cancel():
    """2^-120 (1 + 2^-20) against -2^-120: the difference is the bit that lies below bf16's subnormal numbers."""
    x, dy = torch.zeros(700, 1024, device=DEV), layer(700, 1024, 1024)[1]
    x[0], x[1], dy[0], dy[1] = 2.0 ** -120 * (1 + 2.0 ** -20), -2.0 ** -120, 2.0 ** 100, 2.0 ** 100
    got, want, _ = product(x, dy, 0.0)
    assert bool((want == 2.0 ** -40).all()) and torch.equal(got.double(), want)


def test_products_below_the_subnormal_numbers():
    """Terms of 2^-145 and parts of them far below 2^-149: an fp32 sum of them is off by half of that per term."""
    got, want, _ = product(*layer(700, 1024, 1024, 2.0 ** -75, 2.0 ** -70), 0.0)
    assert (got.double() - want).abs().max().item() <= 700 * 2.0 ** -149


def test_sums_of_one_term():
    """One kept element per column: the product rounded once, 2^-24 of it, and less than 2^-30 for the parts that are added
    up below the first (seven additions at 2^-8 of the product).  1.00ff8p0 has the largest second and third parts."""
    x, dy = torch.zeros(700, 1024, device=DEV), layer(700, 1024, 1024, dy_scale=1.0)[1]
    column = torch.arange(1024, device=DEV)
    x[column % 700, column] = layer(1024, 1, 1)[0][:, 0] + 4.0
    worst = float.fromhex("0x1.00ff8p0")
    x[column[::7] % 700, column[::7]] = worst
    dy[:, ::5] = worst
    dy[dy == 0] = 1.0                              # (two of the numbers drawn)
    got, want, _ = product(x, dy, 1.0 - 1024.5 / x.numel())
    assert int((want != 0).sum()) == want.numel()
    err = ((got.double() - want).abs() / want.abs()).max().item()
    print("thirds one term %.4e" % err, flush=True)
    assert err <= 2.0 ** -24 + 2.0 ** -30

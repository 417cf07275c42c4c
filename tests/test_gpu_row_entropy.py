"""The vocabulary reduction as a call of its own (ec_row_entropy) against the oracle's Eq. 1 and
its closed forms, through the C ABI."""
import math

import numpy as np
import pytest
import torch

import paper_2603_18489_amd as ec
from oracle import entropycache as eco

pytestmark = pytest.mark.gpu


def oracle_stats(z):
    out = np.zeros((z.shape[0], 4))
    for i in range(z.shape[0]):
        tok, conf, H = eco.softmax_stats(z[i].astype(np.float64))
        out[i] = (tok, conf, H, z[i].max())
    return out


@pytest.mark.parametrize("rows,V,pad", [(1, 2, 0), (7, 4096, 0), (32, 126464, 0), (34, 152064, 64),
                                        (128, 5000, 3), (3, 163840, 0), (0, 4096, 0)])
def test_row_entropy_matches_oracle(rows, V, pad):
    rng = np.random.default_rng(rows * 7 + V)
    # rows of different sharpness, one with -inf entries, one with two equal maxima
    z = (rng.standard_normal((rows, V)) * rng.uniform(0.5, 12.0, (rows, 1))).astype(np.float32)
    if rows > 2 and V > 8:
        z[1, ::3] = -np.inf
        z[2, 5] = z[2, V - 3] = z[2].max() + 1.0
    buf = torch.zeros((max(rows, 1), V + pad), dtype=torch.float32, device="cuda")
    zt = buf[:rows, :V]
    zt.copy_(torch.from_numpy(z))
    got = ec.row_entropy(zt).cpu().numpy().astype(np.float64)
    ref = oracle_stats(z)
    assert got.shape == (rows, 4)
    if rows == 0:
        return
    assert np.array_equal(got[:, 0], ref[:, 0])                 # argmax, lowest id on ties
    assert np.array_equal(got[:, 3], ref[:, 3])
    assert np.abs(got[:, 1] - ref[:, 1]).max() <= 4e-6 * ref[:, 1].max()
    assert np.abs(got[:, 2] - ref[:, 2]).max() <= 4e-6 * math.log(V)
    if rows > 2 and V > 8:
        assert int(got[2, 0]) == 5


def test_row_entropy_closed_forms():
    V = 126464
    z = torch.zeros((4, V), dtype=torch.float32, device="cuda")
    z[1] = 3.25                       # uniform at another level: shift invariance
    z[2, :] = -float("inf")
    z[2, 77] = z[2, 99000] = 1.5      # two equal maxima, nothing else: H = ln 2
    z[3, :] = -1e4
    z[3, 123] = 50.0                  # one dominant logit: H = 0, confidence 1
    s = ec.row_entropy(z).cpu().numpy()
    for r in (0, 1):
        assert s[r, 0] == 0 and s[r, 2] == pytest.approx(math.log(V), rel=1e-6)
        assert s[r, 1] == pytest.approx(1.0 / V, rel=1e-6)
    assert s[2, 0] == 77 and s[2, 1] == pytest.approx(0.5, rel=1e-6)
    assert s[2, 2] == pytest.approx(math.log(2.0), rel=1e-6)
    assert s[3, 0] == 123 and s[3, 1] == 1.0 and s[3, 2] == 0.0
    # deterministic: the same input gives the same bits
    assert np.array_equal(s, ec.row_entropy(z).cpu().numpy())


@pytest.mark.parametrize("rows,V,pad", [(1, 2047, 0), (3, 2048, 1), (2, 2049, 0), (5, 16383, 3),
                                        (128, 16384, 0), (4, 16385, 0), (2, 163839, 1)])
def test_row_entropy_part_edges_and_values_without_a_distribution(rows, V, pad):
    """Part boundaries (2048 logits), both sides of the one-launch limit (16384 logits), rows that
    start at any 4-byte address; -inf, NaN and +inf logits.  Bounds as above: float32 sums."""
    rng = np.random.default_rng(V)
    z = (rng.standard_normal((rows, V)) * 6.0).astype(np.float32)
    z[0, 1::2] = -np.inf                      # probability 0
    z[-1, V - 1] = z[-1].max() + 2.0          # the maximum in the last part's tail
    buf = torch.zeros((rows, V + pad), dtype=torch.float32, device="cuda")
    zt = buf[:, :V]
    zt.copy_(torch.from_numpy(z))
    got = ec.row_entropy(zt).cpu().numpy().astype(np.float64)
    ref = oracle_stats(z)
    assert np.array_equal(got[:, 0], ref[:, 0]) and np.array_equal(got[:, 3], ref[:, 3])
    assert np.abs(got[:, 1] / ref[:, 1] - 1.0).max() <= 4e-6
    assert np.abs(got[:, 2] - ref[:, 2]).max() <= 4e-6 * math.log(V)
    zt[0, 5] = float("nan")                   # a NaN: NaN statistics, the others untouched
    s = ec.row_entropy(zt).cpu().numpy()
    assert np.isnan(s[0, 1]) and (rows == 1 or np.array_equal(s[1:], got[1:].astype(np.float32)))
    zt[0, :] = float("nan")                   # no maximum at all: no token either
    s = ec.row_entropy(zt).cpu().numpy()
    assert np.isnan(s[0, 1]) and not 0 <= s[0, 0] < V
    zt[0, :] = -float("inf")                  # one +inf among -inf: certain
    zt[0, V // 2] = float("inf")
    s = ec.row_entropy(zt).cpu().numpy()
    assert s[0, 0] == V // 2 and s[0, 1] == 1.0 and s[0, 2] == 0.0


def test_row_entropy_streams():
    """The default stream, a current side stream and an explicit one give the same bits, also when
    the workspace's memory is handed on to later work right behind the call."""
    z = torch.randn((64, 40000), dtype=torch.float32, device="cuda") * 4.0
    ref = ec.row_entropy(z).cpu().numpy()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = []
        for _ in range(4):
            got.append(ec.row_entropy(z))
            torch.empty(ec.load_library().ec_row_entropy_workspace_bytes(64, 40000),
                        dtype=torch.uint8, device="cuda").fill_(255)
        got = [g.cpu().numpy() for g in got]
    explicit = ec.row_entropy(z, stream=side).cpu().numpy()
    assert all(np.array_equal(g, ref) for g in got) and np.array_equal(explicit, ref)


@pytest.mark.parametrize("side_first", [False, True])
def test_row_entropy_calls_on_two_streams_at_once(side_first):
    """A call on the current stream, still pending, and a call on another stream with logits of its own:
    each gives the bits it gives alone.  (More than 16384 logits: the two-launch form, whose partial
    tuples live in the workspace.)"""
    R, V = 128, 163840
    a = torch.randn((R, V), dtype=torch.float32, device="cuda") * 4.0
    b = torch.randn((R, V), dtype=torch.float32, device="cuda") * 8.0
    ref_a, ref_b = ec.row_entropy(a).cpu().numpy(), ec.row_entropy(b).cpu().numpy()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(4):
        busy = [torch.mul(a, 1.0) for _ in range(3)]      # the current stream is behind
        if side_first:
            got_b = ec.row_entropy(b, stream=side)
            got_a = ec.row_entropy(a)
        else:
            got_a = ec.row_entropy(a)
            got_b = ec.row_entropy(b, stream=side)
        late = got_b * 1.0                                # used on the current stream, then given back
        del got_b
        more = ec.row_entropy(a, stream=side)
        assert np.array_equal(got_a.cpu().numpy(), ref_a)
        assert np.array_equal(late.cpu().numpy(), ref_b)
        assert np.array_equal(more.cpu().numpy(), ref_a)
        del busy


@pytest.mark.parametrize("V", [2048, 4099, 40961])
def test_row_entropy_ties_nan_and_wide_ranges(V):
    """Each row holds its maximum twice, at elements of every distance a wave tells apart (lanes, loads, groups of four
    loads, parts): the lower one is the token.  Logits far below the maximum count nothing, as far as float32 reaches; a
    single NaN among finite logits leaves the maximum and takes the sums."""
    rng = np.random.default_rng(V)
    at = [(i, i + gap) for i in (0, 63, 64, 190, 255, 256, 1983, 2047 - 256) for gap in (1, 64, 128, 256) if i + gap < V]
    z = (rng.standard_normal((len(at) + 3, V)) * 3.0).astype(np.float32)
    for row, (i, j) in enumerate(at):
        z[row, i] = z[row, j] = 40.0
    z[-3] *= np.float32(30.0)                     # differences of hundreds
    z[-2] = -3.0e38
    z[-2, 7], z[-2, V - 2] = 3.0e38, 2.9e38      # a difference past the type's range
    z[-1, V // 2] = np.nan
    got = ec.row_entropy(torch.from_numpy(z).cuda()).cpu().numpy().astype(np.float64)
    ref = oracle_stats(z[:-1])
    assert np.array_equal(got[:-1, 0], ref[:, 0])
    assert np.array_equal(got[:-1, 3], ref[:, 3])
    assert np.allclose(got[:-1, 1], ref[:, 1], rtol=2e-6, atol=0)
    assert np.allclose(got[:-1, 2], ref[:, 2], rtol=1e-5, atol=1e-6)
    assert got[-1, 3] == np.nanmax(z[-1]) and np.isnan(got[-1, 1:3]).any()


@pytest.mark.parametrize("V", [16384, 131072])
def test_row_entropy_errors_have_no_side(V):
    """Rows whose parts of 2048 logits hold one maximum and logits 5 to 8 below it, which make four fifths of the sum, in the
    one-launch and the two-launch form: the errors of 4096 confidences against 64 bits average out.  About a dozen roundings are
    common to all of a row (lane exchanges, merges, the quotient; the sums before them differ from lane to lane): 2^-24 *
    sqrt(12 / 3) = 1.2e-7 r.m.s. at most, 1.9e-9 in the mean; the hardware's 2^t is 3.4e-9 low on average, 2.8e-9 here; four
    times the one and the other make 1e-8.  (Measured: 3.3e-9 and 2.5e-9; an exponential that takes ln 2 for 3.8e-9 more than it
    is: 2.2e-8.)"""
    rows, gen, err = 128, torch.Generator(device="cuda").manual_seed(V), []
    for _ in range(32):
        z = torch.empty((rows, V), device="cuda").uniform_(-8.0, -5.0, generator=gen)
        z[:, 77::2048] = 0.0
        exact = 1.0 / torch.exp(z.double()).sum(dim=1)
        err.append(ec.row_entropy(z)[:, 1].double() / exact - 1.0)
    err = torch.cat(err)
    print(err.mean().item(), err.square().mean().sqrt().item(), err.abs().max().item())
    assert abs(err.mean().item()) < 1e-8


@pytest.mark.parametrize("V", [4096, 16384, 50000, 163840])
def test_row_entropy_of_logits_masked_with_the_lowest_value(V):
    """Whole parts of 2048 logits at the type's lowest finite value (a vocabulary mask), before, behind and around the others, in the
    one-launch and the two-launch form: they have probability 0 and contribute nothing.  Bounds as above."""
    rng = np.random.default_rng(V)
    z = (rng.standard_normal((4, V)) * 2.0).astype(np.float32)
    low = np.finfo(np.float32).min
    z[0, 2048:] = low
    z[1, :V - 1000] = low
    z[2, :V // 4] = z[2, V // 2:] = low
    z[3, :V // 2] = -3.0e37                    # (times 2048 it is past the type's range)
    got = ec.row_entropy(torch.from_numpy(z).cuda()).cpu().numpy().astype(np.float64)
    ref = oracle_stats(z)
    assert np.array_equal(got[:, 0], ref[:, 0]) and np.array_equal(got[:, 3], ref[:, 3])
    assert np.abs(got[:, 1] / ref[:, 1] - 1.0).max() <= 4e-6
    assert np.abs(got[:, 2] - ref[:, 2]).max() <= 4e-6 * math.log(V)

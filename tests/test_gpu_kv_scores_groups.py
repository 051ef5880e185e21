"""Attention logits of grouped query heads (isoq_kv_scores and
isoq_kv_scores_qjl with two or more query heads per key head: the matrix-core
kernel) against the oracle, at the sizes where its tiles end: every width and
bit width, groups around its tiles of 2, 4 and 8 heads, lengths around its
64-key batches and 256-key rounds, odd block sizes, several rounds per
workgroup, codebooks that one set of level digits does not hold, and
non-finite queries.

Tolerances are those of test_gpu_kv_scores.py and test_gpu_kv_scores_qjl.py
(the bound of an fp32 sum of lookups).  The digits stay inside it: a level is
off by at most 2^-23 of itself, the query by 2^-31 of its largest coordinate,
and the int32 sums are exact.
Needs an MI355X."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_28430_amd as iq  # noqa: E402
import test_gpu_kv_scores as plain  # noqa: E402
import test_gpu_kv_scores_qjl as sketch  # noqa: E402

WIDTHS = (64, 80, 96, 128, 160, 192, 256, 512)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("group", [2, 3])
def test_scores_groups_widths(d, bits, group):
    if d == 512 and bits == 3:
        group = 2   # three heads are past the call's limit
    run = (d // 16 + bits + group) % 4
    plain.run_case(("full", "fast", "2d", "8d")[run], d, bits, "f16" if run % 2 else "f32", n_seqs=2, n_q=2 * group,
                   n_kv=2, bs=(16, 7)[run // 2], seq_lens=[330, 65], seed=d + bits + group)


@pytest.mark.parametrize("d,bits", [(128, 3), (80, 3), (192, 4), (256, 2)])
@pytest.mark.parametrize("group", [4, 5, 8, 9])
def test_scores_groups_tiles(d, bits, group):
    plain.run_case("fast", d, bits, "f16", n_seqs=6, n_q=group, n_kv=1, bs=16, seq_lens=[1, 63, 64, 255, 257, 1030],
                   max_len=1025, seed=d + group)


def test_scores_group_single_head_wide():
    """d = 512, 3 and 4 bits: one query head takes the matrix cores too."""
    for bits in (3, 4):
        plain.run_case("full", 512, bits, "f16", n_seqs=2, n_q=2, n_kv=2, bs=16, seq_lens=[700, 33], seed=bits)


def test_scores_groups_several_rounds():
    """Enough workgroups for 1,024 positions each (four rounds of 256 keys)."""
    plain.run_case("fast", 64, 3, "f16", n_seqs=8, n_q=64, n_kv=32, bs=16, seq_lens=[4109] * 7 + [3000], seed=3)


@pytest.mark.parametrize("d,m,bits,group", [(64, 64, 3, 2), (64, 128, 4, 5), (80, 128, 3, 4), (96, 64, 2, 3),
                                            (128, 128, 3, 8), (128, 64, 4, 2), (160, 128, 2, 4), (192, 128, 4, 9),
                                            (256, 64, 3, 4), (512, 64, 4, 1), (512, 64, 2, 2)])
def test_scores_sketch_groups(d, m, bits, group):
    sketch.run_case("full" if bits != 3 else "2d", d, bits, m, "f16", n_seqs=2, n_q=2 * group, n_kv=2, bs=16,
                    seq_lens=[321, 64], seed=d + m + group)


def wide_codebook(bits, ratio):
    """Levels spread over `ratio`."""
    k = 1 << (bits - 1)
    pos = 0.1 * ratio ** (np.arange(k) / (k - 1) - 1.0)
    return np.concatenate([-pos[::-1], pos]).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("bits,ratio", [(2, 3e4), (2, 1e6), (3, 1e3), (3, 1e5), (4, 200.0), (4, 40.0)])
@pytest.mark.parametrize("group", [2, 3, 9])
def test_scores_groups_wide_codebook(monkeypatch, bits, ratio, group):
    """Levels that one set of digits does not hold: further sets hold them, also
    for a key made of small levels only."""
    k = 1 << (bits - 1)
    levels = wide_codebook(bits, ratio)
    monkeypatch.setattr(oracle, "codebook", lambda b, d: levels)
    plain.run_case("full", 128, bits, "f16", n_seqs=1, n_q=2 * group, n_kv=2, bs=16, seq_lens=[300], seed=bits)
    small = lambda s, h, n: (np.full((n, 128), k, np.uint8), np.ones(n, np.float32))  # noqa: E731
    plain.run_case("full", 128, bits, "f32", n_seqs=1, n_q=2 * group, n_kv=2, bs=16, seq_lens=[70], seed=bits,
                   keys=small)


@pytest.mark.parametrize("d,bits,ratio", [(d, b, None) for d in (64, 128, 192, 256) for b in (2, 3, 4)] +
                         [(128, 2, 1e6), (128, 3, 1e5), (64, 4, 200.0)])
def test_scores_groups_small_level_keys(monkeypatch, d, bits, ratio):
    """Keys made of the two smallest levels +-c only: their logits are exactly
    proportional to c, so they are off by what c is off (2^-23 of itself at
    most) and by the fp32 roundings of the query, of the sum and of its two
    factors (2^-24 each, 2^-22 together)."""
    if ratio:
        monkeypatch.setattr(oracle, "codebook", lambda b, d: wide_codebook(bits, ratio))
    p, rot, levels = plain.make("fast", d, bits, 2)
    half = 1 << (bits - 1)
    rng = np.random.default_rng(d + bits)
    keys = lambda s, h, n: (rng.integers(half - 1, half + 1, (n, d)).astype(np.uint8),  # noqa: E731
                            rng.uniform(0.5, 2.0, n).astype(np.float32))
    cache = plain.Cache(rng, d, bits, 1, 2, 16, [400], keys=keys)
    q = rng.standard_normal((1, 4, d)).astype(np.float32)
    rec, rho, table, lens = cache.device()
    got = iq.isoq_kv_scores(p, torch.from_numpy(q).cuda(), rec, rho, table, lens, 1.0)[0, :, :400].cpu().numpy()
    exp = plain.expected("fast", d, bits, rot, np.float32(levels), 2, q, cache, 1.0, 2)
    ref = np.stack([exp[0, hq][0] for hq in range(4)])
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 2.0 ** -23 + 2.0 ** -22, err * 2.0 ** 24


@pytest.mark.parametrize("ratio", [None, 1e5])
def test_scores_groups_codebook_scale(ratio):
    """Codebooks near the ends of the range of floats (one and several sets of
    digits): the logits of a codebook times a power of two are the logits times
    that power, bit for bit."""
    d, bits = 128, 3
    levels = np.float32(oracle.codebook(bits, d)).astype(np.float64)
    if ratio:
        levels = wide_codebook(bits, ratio)
    rng = np.random.default_rng(9)
    cache = plain.Cache(rng, d, bits, 1, 2, 16, [200])
    rec, rho, table, lens = cache.device()
    q = torch.from_numpy(rng.standard_normal((1, 6, d)).astype(np.float16)).cuda()
    rot = plain.make("full", d, bits, 2)[1]
    got = [iq.isoq_kv_scores(iq.isoq_params_init("full", d, bits, 2, rot=rot, codebook=levels * 2.0 ** e), q, rec, rho,
                             table, lens, 1.0)[0, :, :200].double() * 2.0 ** -e for e in (0, -108, 115)]
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    assert got[0].abs().min() > 0


@pytest.mark.parametrize("d,bits,group,m", [(128, 3, 4, 0), (64, 4, 2, 64), (80, 3, 5, 128), (256, 2, 9, 0),
                                            (96, 4, 3, 64)])
def test_scores_groups_nonfinite_query(d, bits, group, m):
    """A query with an infinity or NaN gives the logits that it gives as the
    only head of its key head (infinite or NaN as IEEE sums are), the group's
    other heads theirs; with and without the filling of positions that have no
    key (a block-table entry out of range, past a length)."""
    rng = np.random.default_rng(5)
    p, rot, levels = plain.make("fast", d, bits, 2)
    sk = iq.isoq_sketch_init(p, m) if m else None
    cache = plain.Cache(rng, d, bits, 2, 2, 16, [300, 41])
    cache.table[0, 3] = -1
    rec, rho, table, lens = cache.device()
    q = rng.standard_normal((2, 2 * group, d)).astype(np.float32)
    kw = {}
    if m:
        kw = dict(sketch=sk, k_gamma=rho * 0.2, k_signs=torch.from_numpy(
            rng.integers(0, 256, tuple(rho.shape) + (m // 8,), dtype=np.uint8)).cuda())

    def scores(rows, **more):
        return iq.isoq_kv_scores(p, torch.from_numpy(np.ascontiguousarray(rows)).cuda(), rec, rho, table, lens, 1.0,
                                 **kw, **more)

    ref = scores(q)
    bad = q.copy()
    bad[0, 1, 5], bad[0, 2 * group - 1, d - 1], bad[1, 0, 3] = np.inf, np.nan, -np.inf
    odd = {(0, 1), (0, 2 * group - 1), (1, 0)}
    got = scores(bad)
    plain_out = torch.full_like(got, float("-inf"))
    scores(bad, scores=plain_out)
    assert torch.equal(torch.nan_to_num(got, nan=7.5), torch.nan_to_num(plain_out, nan=7.5))
    infinite = 0
    for s in range(2):
        for hq in range(2 * group):
            if (s, hq) not in odd:
                assert torch.equal(got[s, hq], ref[s, hq])
                continue
            one = bad[:, [hq % group, group + hq % group]]   # the head as the only one of each key head
            exp = scores(one)[s, hq // group]
            assert torch.equal(torch.nan_to_num(got[s, hq], nan=7.5), torch.nan_to_num(exp, nan=7.5)), (s, hq)
            infinite += int(torch.isposinf(exp).sum())
    assert m or infinite > 0   # (with a sketch, S q is infinite throughout and its +- sums NaN)

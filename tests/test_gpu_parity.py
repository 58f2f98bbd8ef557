"""Parity of the HIP path (through the C ABI) against the CPU float64 oracle.

Rules: kept count and kept index set are exact when the oracle's selection is
fed the GPU's own fp32 scores; scores within 1e-9 + 1e-5*value (either input
dtype: the oracle sees the exact device inputs); attention outputs within max-abs 2e-2
(bf16) / 1e-4 (fp32) with the oracle evaluated on the GPU's index set;
compaction bit-exact.
"""
import math
import sys

import numpy as np
import pytest
import torch

import paper_2410_08584_amd as z
from oracle import zipvl_oracle as oz
from workloads import hybrid_probes, make_custom, make_workload

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ATOL_OUT = {"f32": 1e-4, "bf16": 2e-2}


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def dev(x32: np.ndarray, dtype: str) -> torch.Tensor:
    t = torch.from_numpy(np.ascontiguousarray(x32)).to(DEV)
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def host64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def score_tol(dtype):
    # The oracle is fed the exact device inputs, so bf16 storage adds nothing: products of bf16 values are
    # exact in fp32 and both dtypes accumulate in fp32.  Relative error of a probability = ln 2 x the absolute
    # error of its log2-domain exponent (about 2e-6 at |logit| <= 30) plus one ulp each for exp2 and log2.
    return (1e-9, 1e-5)


WORST_SCORE_ERR = {"rel": 0.0}       # largest |got - ref| / (1e-9/1e-5 + |ref|) seen in this process, for the log


def assert_scores_close(got, ref, dtype, what):
    a, r = score_tol(dtype)
    err = np.abs(got - ref) - (a + r * np.abs(ref))
    WORST_SCORE_ERR["rel"] = max(WORST_SCORE_ERR["rel"], float((np.abs(got - ref) / (a / r + np.abs(ref))).max()))
    assert err.max() <= 0, f"{what}: worst excess {err.max():.3e} at {np.unravel_index(err.argmax(), err.shape)}"


# ------------------------------------------------------------------ compaction
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)])
def test_compact_kv_bit_exact(dtype, d):
    say(f"compact_kv dtype={dtype} d={d}")
    B, Hkv, n, cap = 2, 3, 333, 300
    r = np.random.Generator(np.random.PCG64(5))
    w = make_custom(B, Hkv, Hkv, n, d, dtype, seed=11)
    # token-major memory order [B,n,H,d] viewed as [B,H,n,d]
    K = dev(w.K, dtype).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    V = dev(w.V, dtype)
    ks = [1, 64, 65, 300, 7, 129]
    idx = np.zeros((B * Hkv, n), dtype=np.int32)
    for u, k in enumerate(ks):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    Kc, Vc, ln = z.zipvl_compact_kv(K, V, torch.from_numpy(idx).to(DEV),
                                    torch.tensor(ks, dtype=torch.int32, device=DEV), cap)
    torch.cuda.synchronize()
    assert ln.cpu().tolist() == ks
    Kc_h, Vc_h = Kc.to(torch.float32).cpu().numpy(), Vc.to(torch.float32).cpu().numpy()
    for u, k in enumerate(ks):
        b, g = divmod(u, Hkv)
        ko, vo, _ = oz.compact_kv(w.K[b, g], w.V[b, g], idx[u, :k])
        assert Kc_h[u, :k].tobytes() == ko.tobytes() and Vc_h[u, :k].tobytes() == vo.tobytes()
    # all rows, and a cap smaller than k
    Kc2, Vc2, ln2 = z.zipvl_compact_kv(K, V, None, None, 100)
    torch.cuda.synchronize()
    assert ln2.cpu().tolist() == [100] * (B * Hkv)
    assert Kc2.to(torch.float32).cpu().numpy()[4].tobytes() == w.K[1, 1, :100].tobytes()


# ------------------------------------------------------------------ selection
SELECT_WS = {}


def _select_case(name, mass, rank, tau):
    say(f"select case={name} units={mass.shape[0]} n={mass.shape[1]} tau={tau}")
    mass = np.ascontiguousarray(mass)
    rank = None if rank is None else np.ascontiguousarray(rank)
    m_d = torch.from_numpy(mass).to(DEV)
    r_d = None if rank is None else torch.from_numpy(rank).to(DEV)
    units = mass.shape[0]
    ws = SELECT_WS.setdefault(units, z.select_workspace(units, DEV))      # reused across cases: every call must leave it zero
    ref = [oz.select(mass[u], None if rank is None else rank[u], tau) for u in range(units)]
    long = mass.shape[1] > 32768                              # shorter vectors: keys in registers, and the workspace is not used
    for form, w_ in (("one kernel" if long else "registers", None), ("two kernels" if long else "registers, workspace given", ws)):
        idx, k = z.zipvl_select(m_d, r_d, tau, ws=w_)
        torch.cuda.synchronize()
        idx, k = idx.cpu().numpy(), k.cpu().numpy()
        for u in range(units):
            p, T = ref[u]
            assert k[u] == p, f"{name} ({form}) unit {u}: k {k[u]} != {p}"
            assert np.array_equal(idx[u, :p], T), f"{name} ({form}) unit {u}: index set differs"
    assert int(ws.view(torch.int32).abs().sum().item()) == 0, f"{name}: the workspace was not left zero"


def test_select_exact_on_synthetic_distributions():
    r = np.random.Generator(np.random.PCG64(21))

    def norm(x):
        return (x / x.sum(axis=1, keepdims=True)).astype(np.float32)

    for n in (1, 2, 63, 64, 65, 577, 1024, 4097, 18432):
        skew = norm(r.random((3, n)) ** 8 + 1e-9)
        rk = (skew * (1 + 0.5 * r.random((3, n)))).astype(np.float32)
        _select_case(f"skew-n{n}", skew, rk, 0.975)
        _select_case(f"skew-single-n{n}", skew, None, 0.9)
    # around the block of keys that the kernels for long vectors stage in LDS (27648), and such vectors themselves (> 32768)
    for n in (27648, 27649, 131072):
        big = norm(r.random((2, n)) ** 6 + 1e-9)
        _select_case(f"long-n{n}", big, (big * (1 + r.random((2, n)))).astype(np.float32), 0.975)
        _select_case(f"long-single-n{n}", big, None, 0.95)
    n = 3000
    ties = norm(np.round(r.random((2, n)) * 6) + 1.0)            # 7 distinct values: many ties
    _select_case("ties", ties, ties[:, ::-1].copy(), 0.7)
    _select_case("ties-single", ties, None, 0.6180339887)
    uni = np.full((2, 1000), 2.0 ** -10, dtype=np.float32)
    for tau in (0.5, 0.975, 0.999, 1.0):
        _select_case("uniform", uni, None, tau)
    _select_case("zeros", np.zeros((2, 500), dtype=np.float32), None, 0.9)
    onehot = np.zeros((2, 700), dtype=np.float32); onehot[0, 699] = 1.0; onehot[1, 0] = 1.0
    _select_case("onehot", onehot, None, 0.99)
    tiny = norm(r.random((2, 2048))) * np.float32(2.0 ** -30)      # most values below the 2^-40 grid step
    _select_case("tiny", tiny.astype(np.float32), None, 0.95)
    wide = norm(np.exp(r.normal(0, 6, (4, 8192))))                # many exponents
    for tau in (0.3, 0.95, 0.975, 0.99, 0.99999):
        _select_case("lognormal", wide, (wide * r.random((4, 8192))).astype(np.float32), tau)
    # softmax-like: a few heavy tokens and a long tail, rank boosts the last 64 columns
    tail = norm(np.concatenate([r.random((2, 40)) * 50, r.random((2, 18392)) * 0.01], axis=1))
    rk = tail.copy(); rk[:, -64:] *= np.linspace(1, 64, 64, dtype=np.float32)
    _select_case("heavy+tail", tail, rk, 0.975)
    # one first-digit bin (a sixteenth of a binade) holding more elements than the list of candidates takes (1024 of keys in
    # registers; the 2048 of the two-kernel form: below, at its sizes)
    for cnt in (1024, 1025, 2048, 2049, 5000):
        band = (1.0 + r.random((2, cnt)) / 17.0).astype(np.float32)        # all in [1, 1 + 1/16): one bin
        rest = (r.random((2, 3000)) * 0.9).astype(np.float32)
        x = norm(np.concatenate([rest, band], axis=1)[:, r.permutation(3000 + cnt)])
        _select_case(f"crowded-bin-{cnt}", x, (x * (1 + 0.01 * r.random(x.shape))).astype(np.float32), 0.6)
        _select_case(f"crowded-bin-single-{cnt}", x, None, 0.5)
    dup = norm(np.repeat(r.random((2, 40)) ** 3, 100, axis=1)[:, r.permutation(4000)])      # 40 distinct values, 100 copies each
    _select_case("blocks-of-equal-values", dup, dup[:, ::-1].copy(), 0.8)


@pytest.mark.parametrize("n", [1, 2, 64, 1023, 1024, 1025, 2048, 3073, 6144, 6145, 12289, 20480, 24577, 28673, 32767, 32768, 32769])
def test_select_with_keys_in_registers_at_the_edges_of_its_sizes(n):
    """Either side of every number of keys per thread, and of the largest; scores far above and far below the octaves that
    the first digit covers, more equal or nearly equal scores than the list of candidates holds, and ranks of zero that
    the set has to reach down to."""
    r = np.random.Generator(np.random.PCG64(n))
    x = np.exp(r.normal(0, 2.2, (2, n)))
    x = (x / x.sum(axis=1, keepdims=True)).astype(np.float32)
    rk = (x * (1 + r.random((2, n)))).astype(np.float32)
    _select_case(f"registers-n{n}", x, rk, 0.975)
    _select_case(f"registers-low-n{n}", (x * np.float32(2.0 ** -12)).astype(np.float32), (rk * np.float32(2.0 ** -40)).astype(np.float32), 0.9)
    _select_case(f"registers-high-n{n}", x, (rk * np.float32(2.0 ** 60)).astype(np.float32), 0.5)
    near = (np.float32(1.0 / n) * (1 + r.integers(0, 50, (2, n)) * 2.0 ** -20)).astype(np.float32)
    _select_case(f"registers-near-n{n}", near, near[:, ::-1].copy(), 0.6)
    holes = np.where(r.random((2, n)) < 0.9, 0, rk).astype(np.float32)
    _select_case(f"registers-holes-n{n}", x, holes, 0.975)


@pytest.mark.parametrize("n", [32769, 33000, 60000])
def test_select_of_long_vectors(n):
    """n > 32768: one kernel that re-reads the vectors, and two kernels with a workspace.  Nothing to sum, every token, one token, few
    values, close values, a first-digit bin that holds as many keys as the gathered list takes (2048) and more, scores far
    outside the octaves of a softmax."""
    r = np.random.Generator(np.random.PCG64(n))
    norm = lambda x: (x / x.sum(axis=1, keepdims=True)).astype(np.float32)
    x = norm(np.exp(r.normal(0, 2.2, (2, n))))
    rk = (x * (1 + r.random((2, n)))).astype(np.float32)
    for tau in (1e-9, 0.5, 0.99999, 1.0):
        _select_case(f"long-tau-n{n}", x, rk, tau)
    zeros = np.zeros((2, n), dtype=np.float32)
    _select_case(f"long-zeros-n{n}", zeros, None, 0.9)
    _select_case(f"long-zeros-ranked-n{n}", zeros, rk, 0.9)
    _select_case(f"long-rank-zeros-n{n}", x, zeros, 0.9)
    onehot = zeros.copy()
    onehot[0, n - 1] = onehot[1, 0] = 1.0
    _select_case(f"long-onehot-n{n}", onehot, None, 0.99)
    _select_case(f"long-uniform-n{n}", np.full((2, n), 2.0 ** -17, dtype=np.float32), None, 0.5)
    few = norm(np.round(r.random((2, n)) * 6) + 1.0)
    _select_case(f"long-few-values-n{n}", few, few[:, ::-1].copy(), 0.7)
    near = (np.float32(1.0 / n) * (1 + r.integers(0, 50, (2, n)) * 2.0 ** -20)).astype(np.float32)
    _select_case(f"long-near-n{n}", near, near[:, ::-1].copy(), 0.6)
    holes = np.where(r.random((2, n)) < 0.9, 0, rk).astype(np.float32)
    _select_case(f"long-holes-n{n}", x, holes, 0.975)
    _select_case(f"long-wide-n{n}", (x * np.float32(2.0 ** -12)).astype(np.float32), (rk * np.float32(2.0 ** 60)).astype(np.float32), 0.9)
    for cnt in (2047, 2048, 2049, 5000):
        band = (1.0 + r.random((2, cnt)) / 17.0).astype(np.float32)        # all in [1, 1 + 1/16): one bin
        y = norm(np.concatenate([r.random((2, n - cnt)) * 0.02, band], axis=1)[:, r.permutation(n)])
        _select_case(f"long-crowded-bin-{cnt}-n{n}", y, (y * (1 + 0.01 * r.random(y.shape))).astype(np.float32), 0.6)
        _select_case(f"long-crowded-bin-single-{cnt}-n{n}", y, None, 0.5)


@pytest.mark.parametrize("n", [5000, 33000])
def test_select_status_word_reports_inputs_outside_the_contract(n):
    """The optional status word: 0 for valid input, and one bit each for a sign-bit entry, a non-finite entry and a
    mass that sums to 2 or more; with and without a workspace, at a size of either dispatch; the selection itself still runs
    (and, for the sign-bit case, treats the entry as zero: the result equals the oracle's on the cleaned vector)."""
    say(f"select status word n={n}")
    r = np.random.Generator(np.random.PCG64(23))
    good = r.random((5, n)).astype(np.float32) ** 4
    good /= good.sum(axis=1, keepdims=True)
    x = np.ascontiguousarray(good.astype(np.float32))
    x[1, 17] = -x[1, 17]                         # negative entry
    x[2, 4000] = np.float32("inf")               # infinity in mass
    x[3] *= np.float32(2.5)                      # sums to 2.5: the integer sum no longer fits its field
    rk = np.ascontiguousarray((good * (1 + r.random((5, n)))).astype(np.float32))
    rk[4, 99] = np.float32("nan")                # NaN in rank only
    ws = z.select_workspace(5, DEV)
    expect = [0, z.SELECT_NEGATIVE, z.SELECT_NONFINITE, z.SELECT_OVERFLOW, z.SELECT_NONFINITE]
    for w_ in (None, ws):
        st = torch.full((5,), -1, dtype=torch.int32, device=DEV)
        idx, k = z.zipvl_select(torch.from_numpy(x).to(DEV), torch.from_numpy(rk).to(DEV), 0.9, ws=w_, status=st)
        torch.cuda.synchronize()
        assert st.cpu().tolist() == expect, st.cpu().tolist()
        for u in (0, 1):                         # valid unit, and the unit whose negative entry counts as zero
            clean = np.where(np.signbit(x[u]), np.float32(0), x[u])
            p, T = oz.select(clean, rk[u], 0.9)
            assert int(k[u]) == p and np.array_equal(idx[u, :p].cpu().numpy(), T)
    # without a status word nothing is written and valid input gives the same result
    idx2, k2 = z.zipvl_select(torch.from_numpy(x[:1]).to(DEV), torch.from_numpy(rk[:1]).to(DEV), 0.9)
    torch.cuda.synchronize()
    assert int(k2[0]) == int(k[0]) and torch.equal(idx2[0, :int(k2[0])], idx[0, :int(k2[0])])


@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 127, 128])
def test_rank_divides_by_the_probes_at_or_after_each_key(m):
    """Eq. (8)'s count for every key of a 300-token unit, with probes scattered over it (first key a probe, last not):
    mass and rank come from one sum, so rank * count = mass * m up to two roundings."""
    say(f"score rank counts m={m}")
    n = 300
    r = np.random.Generator(np.random.PCG64(m))
    pos = np.sort(np.concatenate([[0], 1 + r.permutation(n - 3)[: m - 1]])) if m > 1 else np.array([137])
    w = make_custom(1, 2, 1, n, 64, "f32", seed=73, m=64)
    mass, rank = z.zipvl_score(dev(w.Q, "f32"), dev(w.K, "f32"), pos, w.scale)
    torch.cuda.synchronize()
    cnt = (pos[:, None] >= np.arange(n)[None, :]).sum(axis=0)
    a, b = host64(mass)[0] * m, host64(rank)[0] * cnt
    assert (host64(rank)[0][cnt == 0] == 0).all() and (host64(mass)[0][cnt == 0] == 0).all()
    assert (np.abs(a - b) <= 4 * 2.0 ** -24 * a).all()


def test_scores_per_query_head_are_the_single_head_scores():
    """ZIPVL_SCORE_PER_QHEAD: one row per query head, nothing averaged (the paper's single-head equations); the group
    mean of those rows is what the default mode returns."""
    say("score per query head")
    B, Hq, Hkv, n, d, dtype = 2, 6, 2, 777, 128, "bf16"
    G = Hq // Hkv
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=19)
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    mass_h, rank_h = z.zipvl_score(Q, K, w.probe_pos, w.scale, flags=z.SCORE_PER_QHEAD)
    mass_g, rank_g = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    torch.cuda.synchronize()
    assert mass_h.shape == (B * Hq, n) and mass_g.shape == (B * Hkv, n)
    mh, rh = host64(mass_h).reshape(B, Hq, n), host64(rank_h).reshape(B, Hq, n)
    for b in range(B):
        for h in range(Hq):
            mo, ro = oz.token_scores(w.Q[b, h:h + 1], w.K[b, h // G:h // G + 1], w.probe_pos, w.scale)    # one head, its own KV head
            assert_scores_close(mh[b, h][None], mo, dtype, "mass")
            assert_scores_close(rh[b, h][None], ro, dtype, "rank")
    np.testing.assert_allclose(mh.reshape(B, Hkv, G, n).mean(axis=2), host64(mass_g).reshape(B, Hkv, n), rtol=2e-6, atol=1e-12)


# ------------------------------------------------------------------ scores
SCORE_CASES = [
    # B, Hq, Hkv, n, d, dtype, m, probe
    (1, 4, 4, 576, 64, "f32", 64, None),
    (2, 4, 2, 700, 128, "bf16", 64, None),
    (1, 6, 2, 333, 64, "bf16", 24, None),
    (1, 2, 1, 1500, 128, "f32", 64, None),
    (1, 7, 1, 2100, 128, "bf16", 64, "scattered"),
    (1, 2, 2, 70, 64, "f32", 64, None),
    (1, 4, 2, 1500, 128, "bf16", 128, "hybrid"),
    (1, 2, 2, 900, 64, "f32", 100, "hybrid"),
    (1, 3, 1, 640, 64, "bf16", 128, "hybrid"),
    (1, 2, 1, 700, 128, "f32", 128, "hybrid"),
]


@pytest.mark.parametrize("case", SCORE_CASES, ids=lambda c: f"B{c[0]}Hq{c[1]}Hkv{c[2]}n{c[3]}d{c[4]}{c[5]}m{c[6]}{c[7] or ''}")
def test_scores_match_oracle(case):
    B, Hq, Hkv, n, d, dtype, m, probe = case
    say(f"score case={case}")
    pp = None
    if probe == "scattered":
        r = np.random.Generator(np.random.PCG64(3))
        pp = np.sort(np.concatenate([r.choice(n - 200, m - 20, replace=False), np.arange(n - 20, n)])).astype(np.int32)
    if probe == "hybrid":
        pp = hybrid_probes(n, seed=n, recent=64, random=m - 64)
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=100 + n, m=m, probe_pos=pp)
    assert len(w.probe_pos) == m
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    torch.cuda.synchronize()
    mass, rank = host64(mass).reshape(B, Hkv, n), host64(rank).reshape(B, Hkv, n)
    for b in range(B):
        mo, ro = oz.token_scores(w.Q[b], w.K[b], w.probe_pos, w.scale)
        assert_scores_close(mass[b], mo, dtype, "mass")
        assert_scores_close(rank[b], ro, dtype, "rank")
        np.testing.assert_allclose(mass[b].sum(axis=1), 1.0, atol=2e-5)
    say(f"  worst relative score error so far {WORST_SCORE_ERR['rel']:.2e} (bound 1e-5)")


@pytest.mark.parametrize("dtype,d,G,Hkv,n,m", [("bf16", 128, 5, 1, 90, 40), ("bf16", 128, 8, 2, 40, 40), ("f32", 64, 9, 1, 1000, 64), ("bf16", 64, 11, 1, 700, 96),
                                               ("bf16", 128, 16, 1, 150, 128), ("f32", 128, 16, 1, 500, 65), ("bf16", 128, 8, 1, 17000, 33), ("bf16", 64, 13, 1, 9000, 128),
                                               ("f32", 64, 7, 16, 2880, 128), ("f32", 128, 5, 60, 360, 128), ("f32", 128, 7, 2, 500, 128)])
def test_scores_of_wide_groups(dtype, d, G, Hkv, n, m):
    """More (head, block of 32 probes) tasks than one workgroup of the row statistics takes, 8 or 4 a workgroup, in even and uneven
    shares, over few and many keys, in one turn of the chip and (fp32, 16 and 60 KV heads) in two: the oracle's scores with the bound above, for
    probes over the whole sequence."""
    say(f"scores of wide groups dtype={dtype} d={d} G={G} n={n} m={m}")
    r = np.random.Generator(np.random.PCG64(81))
    pp = np.sort(np.append(r.choice(n - 1, m - 1, replace=False), n - 1)).astype(np.int32)
    w = make_custom(1, G * Hkv, Hkv, n, d, dtype, seed=82, m=m, probe_pos=pp)
    mass, rank = z.zipvl_score(dev(w.Q, dtype), dev(w.K, dtype), w.probe_pos, w.scale)
    torch.cuda.synchronize()
    mo, ro = oz.token_scores(w.Q[0], w.K[0], w.probe_pos, w.scale)
    assert_scores_close(host64(mass), mo, dtype, "mass")
    assert_scores_close(host64(rank), ro, dtype, "rank")


# chunks of 2, 3, 8, 9 and more stages with 8 waves (scores stage by stage up to 2, eight stages at a time from 3 on), rounds of 16 waves
@pytest.mark.parametrize("dtype,d,Hq,Hkv,n,m", [("bf16", 64, 32, 32, 4096, 64), ("bf16", 64, 32, 32, 4097, 64), ("bf16", 64, 128, 128, 4096, 64), ("bf16", 64, 128, 128, 4200, 64),
                                                ("bf16", 128, 32, 32, 2048, 128), ("bf16", 128, 32, 32, 2049, 128), ("bf16", 64, 128, 128, 8300, 128), ("f32", 64, 128, 128, 2100, 96),
                                                ("bf16", 64, 36, 4, 3000, 64), ("bf16", 128, 36, 4, 3000, 64)])
def test_scores_of_chunks_of_few_and_many_stages(dtype, d, Hq, Hkv, n, m):
    """The last 32 and random probe rows against the oracle, in the first, a middle and the last KV head."""
    say(f"score {dtype} d={d} Hq={Hq} Hkv={Hkv} n={n} m={m}")
    G, gen = Hq // Hkv, torch.Generator(device=DEV)
    gen.manual_seed(78)
    Q, K = (torch.randn((1, h, n, d), generator=gen, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32) for h in (Hq, Hkv))
    r = np.random.Generator(np.random.PCG64(79))
    pos = sorted([int(x) for x in r.choice(n - 32, m - 32, replace=False)] + list(range(n - 32, n)))
    mass, rank = z.zipvl_score(Q, K, pos, d ** -0.5)
    torch.cuda.synchronize()
    for g in (0, Hkv // 2, Hkv - 1):
        mo, ro = oz.token_scores(host64(Q[0, g * G : g * G + G]), host64(K[0, g : g + 1]), np.array(pos), d ** -0.5)
        assert_scores_close(host64(mass[g : g + 1]), mo, dtype, "mass")
        assert_scores_close(host64(rank[g : g + 1]), ro, dtype, "rank")


# bytes from a row of Q to the next, rows: 16 MiB and more (addresses of 64 bits), below with rows from 2 GiB on (offsets of 32 bits without a sign), below and 4 GiB in all
@pytest.mark.parametrize("row_bytes,n", [((16 << 20) + 256, 70), (15 << 20, 200), (15 << 20, 290)])
@pytest.mark.parametrize("dtype,d,Hq,Hkv", [("bf16", 128, 4, 2), ("bf16", 128, 10, 1), ("f32", 128, 3, 3), ("f32", 128, 10, 1), ("f32", 64, 4, 4), ("bf16", 64, 2, 2)])
def test_scores_of_queries_in_rows_far_apart(dtype, d, Hq, Hkv, row_bytes, n):
    """Probe rows of a Q whose rows lie up to 4 GiB and further from its first one: bit for bit the scores of the contiguous Q."""
    say(f"score {dtype} d={d} Hq={Hq} Hkv={Hkv} n={n} rows {row_bytes} bytes apart")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(83)
    Q, K = (torch.randn((1, h, n, d), generator=gen, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32) for h in (Hq, Hkv))
    stride = row_bytes // Q.element_size()
    far = torch.empty((n * stride,), dtype=Q.dtype, device=DEV).as_strided((1, Hq, n, d), (0, d, stride, 1))
    far.copy_(Q)
    r = np.random.Generator(np.random.PCG64(84))
    pos = sorted([0, n - 1] + [int(x) for x in r.choice(np.arange(1, n - 1), 57, replace=False)])
    near = z.zipvl_score(Q, K, pos, d ** -0.5)
    got = z.zipvl_score(far, K, pos, d ** -0.5)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(near, got)) and bool((got[0] > 0).all())


@pytest.mark.parametrize("dtype,d,Hq,Hkv,n", [("bf16", 128, 4, 4, 1500), ("bf16", 64, 28, 4, 700), ("f32", 64, 4, 2, 333), ("f32", 128, 20, 2, 200)])
def test_scores_of_rows_whose_sums_do_not_fit_one_number(dtype, d, Hq, Hkv, n):
    """Sums of exp2 beyond 2^100 and below 2^-100, in some chunks, rows and heads and not in others, and a row that is not a number.
    A log2-domain exponent x carries sqrt(d) 2^-24 |x| < 1e-6 |x| from the fp32 product sum and its roundings."""
    say(f"score {dtype} d={d} Hq={Hq} Hkv={Hkv} n={n}, large logits")
    w = make_custom(1, Hq, Hkv, n, d, dtype, seed=77, m=64)
    G, K32, Q32 = Hq // Hkv, w.K.copy(), w.Q.copy()
    last = Q32[:, ::G, n - 1] / np.linalg.norm(Q32[:, ::G, n - 1], axis=-1, keepdims=True)
    K32[:, :, n // 3] += 60 * last                             # one key far above the others, in one chunk
    K32[:, 0] -= 40 * last[:, :1]                              # the first KV head: all of them far below zero
    Q32[:, 1::2, n - 64 : n - 40] *= 3
    if Hq > 2:
        Q32[:, 2, n - 20] = 0
    Q, K = dev(Q32, dtype), dev(K32, dtype)
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    torch.cuda.synchronize()
    Qh, Kh = host64(Q)[0], host64(K)[0]
    big = max(np.abs(Qh[h, n - 64:] @ Kh[h // G].T).max() for h in range(Hq)) * w.scale * 1.4427
    say(f"  largest log2-domain logit {big:.0f}")
    assert big > 200
    mo, ro = oz.token_scores(Qh, Kh, w.probe_pos, w.scale)
    for got, ref in ((mass, mo), (rank, ro)):
        assert (np.abs(host64(got) - ref) <= 1e-9 + (1e-5 + 1e-6 * big) * np.abs(ref)).all()
    Q[0, 0, n - 9] = float("nan")                              # a probe row of head 0 only: the other KV heads do not see it
    nan_mass, _ = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    assert torch.equal(nan_mass[1:], mass[1:]) and torch.isnan(nan_mass[0]).any()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", ["first-rows", "block-ends-early", "one-past-a-block", "straddling", "last-row-only"])
def test_scores_where_blocks_of_probes_end(name, dtype):
    """Blocks of 32 probes that see few keys, all keys, none of most tiles, or end on the edge of a 32-key tile; the same
    bound as above."""
    n, tail = 1111, list(range(1111 - 40, 1111))
    pp = {"first-rows": list(range(32)) + [n - 1],                      # a block wholly at the start, one probe in the next
          "block-ends-early": list(range(0, 320, 10)) + list(range(400, 432)) + tail,
          "one-past-a-block": list(range(31, 64)) + list(range(95, 128)),   # nothing past token 127 is seen
          "straddling": [0, 31, 32, 33, 63, 64, 500] + list(range(512, 512 + 64)) + tail,
          "last-row-only": [n - 1]}[name]
    say(f"score blocks case={name} dtype={dtype}")
    w = make_custom(1, 6, 2, n, 128, dtype, seed=len(pp), m=len(pp), probe_pos=np.array(pp, dtype=np.int32))
    mass, rank = z.zipvl_score(dev(w.Q, dtype), dev(w.K, dtype), w.probe_pos, w.scale)
    torch.cuda.synchronize()
    mo, ro = oz.token_scores(w.Q[0], w.K[0], w.probe_pos, w.scale)
    assert_scores_close(host64(mass), mo, dtype, "mass")
    assert_scores_close(host64(rank), ro, dtype, "rank")


# ------------------------------------------------------------------ attention
def _attention_case(B, Hq, Hkv, n, d, dtype, ks, seed=0, flags=0, dense=False, reshape_inputs=None):
    G = Hq // Hkv
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=seed)
    if reshape_inputs is not None:                 # (Q, K) -> (Q', K'), rounded back to the storage type
        q2, k2 = reshape_inputs(w.Q, w.K)
        rnd = (lambda x: torch.from_numpy(x).bfloat16().float().numpy()) if dtype == "bf16" else (lambda x: x.astype(np.float32))
        w.Q, w.K = rnd(np.ascontiguousarray(q2, dtype=np.float32)), rnd(np.ascontiguousarray(k2, dtype=np.float32))
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    units = B * Hkv
    r = np.random.Generator(np.random.PCG64(seed + 1))
    idx = np.zeros((units, n), dtype=np.int32)
    for u in range(units):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    if dense:
        O = z.zipvl_sparse_prefill(Q, K, V, None, None, w.scale)
    else:
        O = torch.full((B, Hq, n, d), 7.0, dtype=Q.dtype, device=DEV)   # poison: dropped rows must be rewritten
        z.zipvl_sparse_prefill(Q, K, V, torch.from_numpy(idx).to(DEV),
                               torch.tensor(ks, dtype=torch.int32, device=DEV), w.scale, flags, O=O)
    torch.cuda.synchronize()
    Oh = host64(O)
    worst = 0.0
    for b in range(B):
        for h in range(Hq):
            g = h // G
            u = b * Hkv + g
            T = np.arange(n) if dense else idx[u, :ks[u]]
            ref = oz.kept_token_attention(w.Q[b, h], w.K[b, g], w.V[b, g], T, w.scale,
                                          compact_out=bool(flags & z.OUT_COMPACT))
            got = Oh[b, h, :len(T)] if flags & z.OUT_COMPACT else Oh[b, h]
            worst = max(worst, np.abs(got - ref).max())
    say(f"  worst |dO| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 129, 200])
def test_attention_in_place_is_attention_over_packed_rows(dtype, d, n):
    """Contiguous rows are read where they are, others through the workspace: the same sums in the same order, so the same
    bits.  Every token kept, and an evicted cache whose rows from k on are NaN; then against the oracle."""
    say(f"attention in place dtype={dtype} d={d} n={n}")
    w = make_custom(1, 4, 2, n, d, dtype, seed=n + d)
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)

    def spread(x):                                          # the same rows, 16 bytes apart
        wide = torch.zeros(x.shape[:-1] + (d + 16 // x.element_size(),), dtype=x.dtype, device=DEV)
        wide[..., :d] = x
        return wide[..., :d]

    dense, packed = z.zipvl_sparse_prefill(Q, K, V, None, None, w.scale), z.zipvl_sparse_prefill(Q, spread(K), spread(V), None, None, w.scale)
    mixed = z.zipvl_sparse_prefill(Q, K, spread(V), None, None, w.scale)
    assert torch.equal(dense, packed) and torch.equal(dense, mixed)
    k = max(1, n - 7)
    Kc, Vc = K.clone(), V.clone()
    Kc[:, :, k:] = float("nan")
    Vc[:, :, k:] = float("nan")
    idx = torch.arange(n, dtype=torch.int32, device=DEV).repeat(2, 1)
    kc = torch.full((2,), k, dtype=torch.int32, device=DEV)
    args = (idx, kc, w.scale, z.OUT_FULL | z.KV_ALREADY_COMPACT)
    evicted = z.zipvl_sparse_prefill(Q, Kc, Vc, *args)
    assert torch.equal(evicted, z.zipvl_sparse_prefill(Q, spread(Kc), spread(Vc), *args))
    torch.cuda.synchronize()
    for h in range(4):
        for got, T in ((dense, np.arange(n)), (evicted, np.arange(k))):
            ref = oz.kept_token_attention(w.Q[0, h], w.K[0, h // 2], w.V[0, h // 2], T, w.scale)
            assert np.abs(host64(got[0, h]) - ref).max() <= ATOL_OUT[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,gain", [(1, 1.0), (33, 1.0), (65, 1.0), (129, 1.0), (200, 1.0), (330, 16.0)])
def test_attention_in_place_with_query_tiles_of_128(dtype, d, n, gain):
    """The same in a batch large enough for tiles of 128 queries (more than 512 of them): every token kept, sequences and kept
    counts that are no multiple of 64, rows from k on NaN; gain 16: logits that take the pass with running maxima."""
    Hq, Hkv, k = 4, 2, max(1, n - 7)
    B = 512 // ((n + 127) // 128 * Hq) + 1
    say(f"attention in place, tiles of 128, dtype={dtype} d={d} n={n} B={B}")
    w = make_custom(1, Hq, Hkv, n, d, dtype, seed=n + d + 1)
    Qh = (w.Q * np.float32(gain)).astype(np.float32)
    if dtype == "bf16":
        Qh = torch.from_numpy(Qh).bfloat16().float().numpy()
    Q, K, V = (dev(x, dtype).repeat(B, 1, 1, 1) for x in (Qh, w.K, w.V))

    def spread(x):                                          # the same rows, 16 bytes apart
        wide = torch.zeros(x.shape[:-1] + (d + 16 // x.element_size(),), dtype=x.dtype, device=DEV)
        wide[..., :d] = x
        return wide[..., :d]

    dense = z.zipvl_sparse_prefill(Q, K, V, None, None, w.scale)
    assert torch.equal(dense, z.zipvl_sparse_prefill(Q, spread(K), spread(V), None, None, w.scale))
    Kc, Vc = K.clone(), V.clone()
    Kc[:, :, k:] = float("nan")
    Vc[:, :, k:] = float("nan")
    idx = torch.arange(n, dtype=torch.int32, device=DEV).repeat(B * Hkv, 1)
    kc = torch.full((B * Hkv,), k, dtype=torch.int32, device=DEV)
    args = (idx, kc, w.scale, z.OUT_FULL | z.KV_ALREADY_COMPACT)
    evicted = z.zipvl_sparse_prefill(Q, Kc, Vc, *args)
    assert torch.equal(evicted, z.zipvl_sparse_prefill(Q, spread(Kc), spread(Vc), *args))
    torch.cuda.synchronize()
    for got, T in ((dense, np.arange(n)), (evicted, np.arange(k))):
        assert torch.equal(got, got[:1].expand_as(got))      # every copy the same bits
        for h in range(Hq):
            ref = oz.kept_token_attention(Qh[0, h], w.K[0, h // 2], w.V[0, h // 2], T, w.scale)
            assert np.abs(host64(got[0, h]) - ref).max() <= ATOL_OUT[dtype]


def test_attention_fp32_small_ragged():
    say("attention fp32 d=64 ragged k")
    _attention_case(1, 4, 4, 576, 64, "f32", [576, 1, 130, 67], seed=1)


def test_attention_bf16_gqa_ragged():
    say("attention bf16 d=128 GQA ragged k")
    _attention_case(2, 6, 2, 700, 128, "bf16", [700, 257, 64, 385], seed=2)


def test_attention_kept_count_on_tile_boundaries():
    say("attention bf16 d=128, k = 128, 256, 384 and n (dropped tail must be cleared)")
    _attention_case(2, 4, 2, 640, 128, "bf16", [128, 256, 384, 640], seed=9)
    _attention_case(1, 2, 2, 384, 64, "f32", [384, 128], seed=10)


def test_attention_bf16_d64_and_fp32_d128():
    say("attention bf16 d=64")
    _attention_case(1, 2, 2, 300, 64, "bf16", [300, 129], seed=3)
    say("attention fp32 d=128")
    _attention_case(1, 2, 1, 260, 128, "f32", [200], seed=4)


def test_attention_dense_mode_equals_dense_oracle():
    say("attention dense (idx=k=NULL)")
    _attention_case(1, 4, 2, 450, 128, "bf16", [450, 450], seed=5, dense=True)
    _attention_case(1, 2, 2, 200, 64, "f32", [200, 200], seed=6, dense=True)


def test_attention_logits_far_from_zero():
    """Rows whose logits leave the range in which exponentials need no offset (the kernel's first pass takes
    exp2 of the scaled logits as they are and repeats a workgroup with running maxima when a row sum leaves
    [2^-64, 2^64]): logits of +-150 and more, logits that are all near -100 or near +100, and a mix of ordinary
    and extreme heads in one launch."""
    say("attention with very large / very negative logits")
    for dtype, d, seed, gain in (("bf16", 128, 31, 40.0), ("f32", 64, 32, 16.0)):   # fp32: +-60, within its 1e-4 bound
        ks = [450, 257, 129, 450]
        _attention_case(1, 4, 4, 450, d, dtype, ks, seed=seed, reshape_inputs=lambda q, k: (q * gain, k))
        shift = 3.0 if d == 128 else 4.5
        _attention_case(1, 4, 4, 450, d, dtype, ks, seed=seed + 2, reshape_inputs=lambda q, k: (q - shift, k + shift))
        _attention_case(1, 4, 4, 450, d, dtype, ks, seed=seed + 4, reshape_inputs=lambda q, k: (q + shift, k + shift))
        def mixed(q, k):
            q = q.copy(); q[:, 1] *= gain; q[:, 2] -= shift; k = k.copy(); k[:, 2] += shift
            return q, k
        _attention_case(1, 4, 4, 450, d, dtype, ks, seed=seed + 6, reshape_inputs=mixed)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("gain", [1.0, 16.0])
def test_attention_with_either_query_tile(dtype, d, gain):
    """The same heads in a small call (query tiles of 64, the keys of a tile split over two waves) and repeated in a batch large
    enough for tiles of 128: kept counts around 32-key blocks and both tiles, dropped rows, and logits (gain 16) that take the
    pass with running maxima.  Both against the oracle with the bounds used above."""
    say(f"attention query tiles dtype={dtype} d={d} gain={gain}")
    n, ks = 330, [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 161, 192, 193, 257, 330]
    Hkv = len(ks)
    w = make_custom(1, Hkv, Hkv, n, d, dtype, seed=51)
    rnd = (lambda x: torch.from_numpy(x).bfloat16().float().numpy()) if dtype == "bf16" else (lambda x: x)
    Qh = rnd((w.Q * np.float32(gain)).astype(np.float32))
    Q, K, V = dev(Qh, dtype), dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(52))
    idx = np.zeros((Hkv, n), dtype=np.int32)
    for u, k in enumerate(ks):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV)
    copies = 512 // (3 * Hkv) + 1                            # 3 tiles of 128 per head: beyond 512 tiles
    for B in (1, copies):
        O = torch.full((B, Hkv, n, d), 7.0, dtype=Q.dtype, device=DEV)
        z.zipvl_sparse_prefill(Q.repeat(B, 1, 1, 1), K.repeat(B, 1, 1, 1), V.repeat(B, 1, 1, 1), idx_d.repeat(B, 1), k_d.repeat(B), w.scale, O=O)
        torch.cuda.synchronize()
        assert torch.equal(O, O[:1].expand_as(O))            # every copy the same bits
        for u in range(Hkv):
            ref = oz.kept_token_attention(Qh[0, u], w.K[0, u], w.V[0, u], idx[u, :ks[u]], w.scale)
            worst = np.abs(host64(O[0, u]) - ref).max()
            assert worst <= ATOL_OUT[dtype], f"B={B} k={ks[u]}: {worst:.3e}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,gain", [(900, 1.0), (900, 16.0), (1100, 1.0)])
def test_attention_query_tile_chosen_by_kept_tokens(d, n, gain):
    """A call whose heads may take either query tile, each by its own count: 64 heads alike in fours, counts around 64-row and
    128-row tiles and around the counts where the choice turns (n = 900: four tiles of 128, 1100: 999 and eight tiles); rows packed,
    and in place in an evicted cache that is NaN from row k on; gain 16: logits that take the pass with running maxima."""
    say(f"attention query tile by kept tokens d={d} n={n} gain={gain}")
    ks = [0, 1, 63, 64, 65, 127, 129, 300, 511, 512, 513, 575, 640, 700, n - 1, n] if n < 1000 else [1, 64, 129, 300, 511, 512, 513, 641, 769, 895, 999, 1000, 1023, 1025, n - 1, n]
    units, B = len(ks), 4
    w = make_custom(1, units, units, n, d, "bf16", seed=53)
    Qh = torch.from_numpy((w.Q * np.float32(gain)).astype(np.float32)).bfloat16().float().numpy()
    Q, K, V = (dev(x, "bf16").repeat(B, 1, 1, 1) for x in (Qh, w.K, w.V))
    r = np.random.Generator(np.random.PCG64(54))
    idx = np.zeros((units, n), dtype=np.int32)
    for u, k in enumerate(ks):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV).repeat(B, 1), torch.tensor(ks, dtype=torch.int32, device=DEV).repeat(B)
    packed, inplace = (torch.full((B, units, n, d), 7.0, dtype=Q.dtype, device=DEV) for _ in range(2))
    z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale, O=packed)
    Kc, Vc, _ = z.zipvl_compact_kv(K, V, idx_d, k_d, n)
    Kc, Vc = Kc.view(B, units, n, d), Vc.view(B, units, n, d)
    for u, k in enumerate(ks):
        Kc[:, u, k:] = float("nan")
        Vc[:, u, k:] = float("nan")
    z.zipvl_sparse_prefill(Q, Kc, Vc, idx_d, k_d, w.scale, z.OUT_FULL | z.KV_ALREADY_COMPACT, O=inplace)
    torch.cuda.synchronize()
    assert torch.equal(packed, inplace) and torch.equal(packed, packed[:1].expand_as(packed))
    for u, k in enumerate(ks):
        ref = oz.kept_token_attention(Qh[0, u], w.K[0, u], w.V[0, u], idx[u, :k], w.scale)
        worst = np.abs(host64(packed[0, u]) - ref).max()
        assert worst <= ATOL_OUT["bf16"], f"k={k}: {worst:.3e}"


@pytest.mark.parametrize("copies,Hq,Hkv,n,d,dtype,shared", [(8, 64, 64, 1100, 64, "bf16", False), (74, 56, 8, 129, 128, "bf16", True), (40, 64, 16, 257, 64, "f32", False),
                                                           (5, 40, 10, 1030, 128, "bf16", True), (3, 14, 7, 700, 128, "bf16", False),
                                                           (71, 3, 3, 1100, 64, "bf16", False), (31, 14, 7, 700, 128, "bf16", False), (2, 8, 8, 8300, 64, "bf16", False)])
def test_attention_schedule(copies, Hq, Hkv, n, d, dtype, shared):
    """Which workgroup takes which tile: more tiles than workgroups (the first three: 9, 2 and 3 tiles of 128 a head), more sets than a
    workgroup reads the counts of (the third), several scheduling groups (of 107 and 106, 109 and 108 KV heads), heads that go round the XCDs (the last), a KV head without a token, heads that keep all; one set per
    KV head and one per batch element, full and compact outputs.  Repeated batch elements give the same bits, the first one agrees
    with the oracle."""
    say(f"attention schedule {copies}x{Hq}/{Hkv} n={n} d={d} {dtype} shared={shared}")
    r = np.random.Generator(np.random.PCG64(61))
    few = min(Hkv, 4)                                        # heads that are computed for the oracle; the others repeat them
    w = make_custom(1, few * Hq // Hkv, few, n, d, dtype, seed=62)
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    reps = (Hkv + few - 1) // few
    Q, K, V = (x.repeat(copies, reps, 1, 1)[:, :h].contiguous() for x, h in ((Q, Hq), (K, Hkv), (V, Hkv)))
    ks = [[n, 1, n // 3, 0], [n // 2], [128, n - 1, 64, n // 5]][1 if shared else copies % 2 * 2][:1 if shared else few]
    idx = np.zeros((len(ks), n), dtype=np.int32)
    for u, k in enumerate(ks):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    times = copies if shared else copies * reps
    idx_d = torch.from_numpy(idx).to(DEV).repeat(times, 1).view(copies, -1, n)[:, :1 if shared else Hkv].reshape(-1, n).contiguous()
    k_d = torch.tensor(ks, dtype=torch.int32, device=DEV).repeat(times).view(copies, -1)[:, :1 if shared else Hkv].reshape(-1).contiguous()
    flag = z.T_PER_BATCH if shared else 0
    O, C = (torch.full((copies, Hq, n, d), 7.0, dtype=Q.dtype, device=DEV) for _ in range(2))
    z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale, flag, O=O)
    z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale, flag | z.OUT_COMPACT, O=C)
    torch.cuda.synchronize()
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(C, C[:1].expand_as(C))
    G = Hq // Hkv
    for h in range(Hq):
        u, f = 0 if shared else h // G % few, h // G % few
        k = ks[u]
        if h >= few * G:
            assert torch.equal(O[0, h], O[0, h % (few * G)])
            continue
        ref = oz.kept_token_attention(w.Q[0, h], w.K[0, f], w.V[0, f], idx[u, :k], w.scale)
        worst = np.abs(host64(O[0, h]) - ref).max()
        assert worst <= ATOL_OUT[dtype], f"head {h}, k={k}: {worst:.3e}"
        assert torch.equal(C[0, h, :k], O[0, h][torch.from_numpy(idx[u, :k]).long().to(DEV)])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("copies,n,ks", [(1, 1, (1, 1)), (1, 33, (32, 33)), (1, 65, (64, 65)), (1, 130, (66, 128)), (1, 300, (31, 130)), (1, 300, (0, 300)), (24, 1090, (65, 1089)), (24, 1090, (1, 700))])
@pytest.mark.parametrize("gain", [1.0, 60.0])
def test_attention_of_queries_in_any_rows(copies, n, ks, d, gain):
    """Query rows at any distance from each other ([B, n, Hq, 2 d] and half of it), in tiles of 64 and of 128 queries with 1 to 128 of them, kept and all;
    with rows that repeat their tiles (gain 60).  The same bits as from contiguous queries, which agree with the oracle."""
    say(f"attention strided queries {copies} n={n} ks={ks} d={d} gain={gain}")
    w = make_custom(1, 4, 2, n, d, "bf16", seed=66)
    Qh, Kh = (torch.from_numpy(x * g).bfloat16().float().numpy() for x, g in ((w.Q, gain), (w.K, 1.0)))
    Q, K, V = (dev(x, "bf16").repeat(copies, 1, 1, 1) for x in (Qh, Kh, w.V))
    far = torch.full((copies, n, 4, 2 * d), float("nan"), dtype=Q.dtype, device=DEV)[..., :d].transpose(1, 2)
    far.copy_(Q)
    r = np.random.Generator(np.random.PCG64(67))
    idx = np.zeros((2, n), dtype=np.int32)
    for u, k in enumerate(ks):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    args = torch.from_numpy(idx).to(DEV).repeat(copies, 1), torch.tensor(ks, dtype=torch.int32, device=DEV).repeat(copies), w.scale
    for a in (args, (None, None, w.scale)):
        O = z.zipvl_sparse_prefill(Q, K, V, *a)
        assert torch.equal(O, z.zipvl_sparse_prefill(far, K, V, *a))
        assert torch.equal(O, O[:1].expand_as(O))
        for h in range(4):
            T = np.arange(n) if a[0] is None else idx[h // 2, :ks[h // 2]]
            ref = oz.kept_token_attention(Qh[0, h], Kh[0, h // 2], w.V[0, h // 2], T, w.scale)
            worst = np.abs(host64(O[0, h]) - ref).max()
            assert worst <= ATOL_OUT["bf16"], f"head {h}: {worst:.3e}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,n,ks", [(1, 97, [97, 33]), (1, 257, [256, 129]), (20, 130, None), (300, 130, None), (100, 161, [100, 1]), (160, 161, [161, 129]), (400, 260, [95, 32])])
def test_attention_fp32_in_three_planes(d, B, n, ks):
    """fp32 attention in all its forms (64 queries by eight waves, by four, 128; chosen by the host and by the kept count), at tiles that
    end early: within 4e-6 of the outputs in 64 bits (2-norm).  A logit of size 5 is a chain of 3 d / 8 sums and rounds by some
    2^-25 sqrt(3 d / 8) of it each, 1e-6 in all, its weight by as much; without one of the last planes it would be 2e-5."""
    say(f"attention fp32 in planes d={d} B={B} n={n} k={ks}")
    w = make_custom(1, 4, 2, n, d, "f32", seed=d + n)
    Q, K, V = (dev(x, "f32").repeat(B, 1, 1, 1) for x in (w.Q, w.K, w.V))
    idx = k = None
    T = [np.arange(n)] * 2
    if ks:
        r = np.random.Generator(np.random.PCG64(n))
        T = [np.sort(r.choice(n, x, replace=False)) for x in ks]
        rows = np.zeros((2, n), dtype=np.int32)
        for g in range(2):
            rows[g, :ks[g]] = T[g]
        idx, k = torch.from_numpy(rows).to(DEV).repeat(B, 1), torch.tensor(ks, dtype=torch.int32, device=DEV).repeat(B)
    O = z.zipvl_sparse_prefill(Q, K, V, idx, k, w.scale)
    torch.cuda.synchronize()
    assert torch.equal(O, O[:1].expand_as(O))
    for h in range(4):
        ref = oz.kept_token_attention(w.Q[0, h], w.K[0, h // 2], w.V[0, h // 2], T[h // 2], w.scale)
        err = np.linalg.norm(host64(O[0, h]) - ref) / np.linalg.norm(ref)
        assert err <= 4e-6, f"head {h}: {err:.2e}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B", [1, 20, 120])
def test_attention_fp32_beyond_the_range_of_the_planes(d, B):
    """Values that three bf16 planes do not hold: a key that no query can see (an infinity, logit -inf), an infinity in V, and one just
    below the largest fp32 number, which rounds to an infinity; in all three forms."""
    n, key, inf_row, big_row = 260, 40, 200, 70
    say(f"attention fp32 beyond the planes d={d} B={B}")
    w = make_custom(1, 4, 2, n, d, "f32", seed=d)
    Qh, Kh, Vh = w.Q.copy(), w.K.copy(), w.V.copy()
    Qh[..., 0] = -np.abs(Qh[..., 0]) - np.float32(0.1)
    Kh[:, :, key, 0] = np.inf
    Vh[:, :, inf_row, 3] = np.inf
    Vh[:, :, big_row, 5] = 3.4e38
    O = z.zipvl_sparse_prefill(*(dev(x, "f32").repeat(B, 1, 1, 1) for x in (Qh, Kh, Vh)), None, None, w.scale)
    torch.cuda.synchronize()
    assert torch.equal(O[1:].isnan(), O[:1].expand_as(O)[1:].isnan()) and torch.equal(O.nan_to_num(), O[:1].expand_as(O).nan_to_num())
    for h in range(4):
        q, k, v = (x.astype(np.float64) for x in (Qh[0, h], Kh[0, h // 2], Vh[0, h // 2]))
        got = host64(O[0, h])
        k[key], v[inf_row, 3] = 0.0, 0.0
        s = np.where(np.tril(np.ones((n, n), dtype=bool)), q @ k.T * w.scale, -np.inf)
        s[:, key] = -np.inf
        p = np.exp(s - s.max(axis=1, keepdims=True))
        ref = p @ v / p.sum(axis=1, keepdims=True)
        assert np.all(got[inf_row:, 3] == np.inf)            # rows before it in its block of 32 keys weigh it with 0: no number
        got[inf_row:, 3], ref[inf_row // 32 * 32:, 3] = 0.0, 0.0
        got[inf_row // 32 * 32:inf_row, 3] = 0.0
        assert np.all(np.abs(got - ref) <= ATOL_OUT["f32"] * np.maximum(1.0, np.abs(ref)))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B", [1, 20, 120])
def test_attention_fp32_keeps_its_precision_at_small_and_large_magnitudes(d, B):
    """Magnitudes at which the last of three bf16 planes ends at bf16's smallest number (2^-133): V small as a whole or in one channel,
    a channel that lives by one key of weight 2^-121, queries small against large keys and the other way round; every output within 4e-6
    of its value in 64 bits, channel by channel (as for ordinary values; the weight: an exponent of -121 and its factor are rounded to
    24 bits, 5e-6 of it).  All three forms."""
    n, key = 260, 40
    say(f"attention fp32 at small and large magnitudes d={d} B={B}")
    w = make_custom(1, 4, 2, n, d, "f32", seed=d + 1)
    mul = lambda x, f: (x.astype(np.float64) * f).astype(np.float32)
    one = w.V.copy()
    one[..., 5] = mul(one[..., 5], 1e-36)
    Qk, Kk, Vk = w.Q.copy(), w.K.copy(), w.V.copy()
    Qk, Kk[..., 0] = mul(Qk, 0.05), 0.0
    Qk[..., 0] = -1.0
    Kk[:, :, key] = 0.0
    Kk[:, :, key, 0] = 84.0 / w.scale
    Vk[..., 7] = 0.0
    Vk[:, :, key, 7] = 1024.0
    cases = [(f"V * {f}", w.Q, w.K, mul(w.V, f), 4e-6) for f in (1e-30, 1e-34, 1e-36, 1e-37)]
    cases += [("one channel of V * 1e-36", w.Q, w.K, one, 4e-6), ("Q * 1e-36, K * 1e36", mul(w.Q, 1e-36), mul(w.K, 1e36), w.V, 4e-6),
              ("Q * 1e36, K * 1e-36", mul(w.Q, 1e36), mul(w.K, 1e-36), w.V, 4e-6), ("one key of weight 2^-121", Qk, Kk, Vk, 1.2e-5)]
    for what, Q, K, V, tol in cases:
        O = z.zipvl_sparse_prefill(*(dev(x, "f32").repeat(B, 1, 1, 1) for x in (Q, K, V)), None, None, w.scale)
        torch.cuda.synchronize()
        assert torch.equal(O, O[:1].expand_as(O))
        for h in range(4):
            ref = oz.kept_token_attention(Q[0, h].astype(np.float64), K[0, h // 2].astype(np.float64), V[0, h // 2].astype(np.float64), np.arange(n), w.scale)
            err = np.linalg.norm(host64(O[0, h]) - ref, axis=0) / np.linalg.norm(ref, axis=0)
            assert err.max() <= tol, f"{what}, head {h}, channel {err.argmax()}: {err.max():.2e}"


def test_attention_compact_output_rows():
    say("attention OUT_COMPACT")
    _attention_case(1, 4, 2, 500, 128, "bf16", [333, 128], seed=7, flags=z.OUT_COMPACT)


@pytest.mark.parametrize("n,d,ks", [(40, 128, [40, 39]), (65, 128, [65, 64]), (129, 64, [129, 1]), (333, 128, [333, 320]), (333, 128, [321, 319]),
                                    (447, 64, [447, 446])])
def test_attention_reads_a_ragged_cache_up_to_its_last_row(n, d, ks):
    """Evicted caches whose last 64-row tile is not full, with kept counts in and next to that tile, read in place; NaN
    beyond k.  Bit for bit the attention that gathers from the whole K, V."""
    say(f"attention KV_ALREADY_COMPACT ragged n={n} d={d} k={ks}")
    B, Hq, Hkv, dtype = 1, 4, 2, "bf16"
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=10, m=min(64, n))
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(11))
    idx = np.zeros((2, n), dtype=np.int32)
    for u in range(2):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV)
    Kc = torch.full((2, n, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    Vc = torch.full((2, n, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    z.zipvl_compact_kv(K, V, idx_d, k_d, n, Kc=Kc, Vc=Vc)
    for flags in (z.OUT_FULL, z.OUT_COMPACT):
        O1, O2 = torch.zeros_like(Q), torch.zeros_like(Q)
        z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale, flags, O=O1)
        z.zipvl_sparse_prefill(Q, Kc.view(B, Hkv, n, d), Vc.view(B, Hkv, n, d), idx_d, k_d, w.scale, flags | z.KV_ALREADY_COMPACT, O=O2)
        torch.cuda.synchronize()
        assert torch.equal(O1, O2) and not torch.isnan(O2.float()).any()


@pytest.mark.parametrize("n,d,dtype,ks,gain", [(448, 128, "bf16", [211, 77], 1.0), (333, 128, "bf16", [130, 129], 1.0), (1000, 128, "bf16", [833, 640], 1.0),
                                               (1024, 64, "bf16", [577, 831], 1.0), (1000, 128, "bf16", [705, 1], 40.0), (129, 64, "f32", [65, 63], 1.0),
                                               (640, 128, "f32", [449, 320], 1.0)])
def test_attention_reads_no_row_at_or_beyond_k(n, d, dtype, ks, gain):
    """An evicted cache of exactly max k rows inside a larger allocation of NaN (rows past a unit's k included): a V row
    read at or beyond k would weigh in as 0 * NaN.  The tile with row k - 1 is the first of its workgroup, a later one,
    one in the kernel's steady state, or whole; gain 40: the pass with running maxima.  Bit for bit the attention that
    gathers from the whole K, V."""
    say(f"attention on a cache of max k rows n={n} d={d} {dtype} k={ks} gain={gain}")
    B, Hq, Hkv, cap, guard = 1, 4, 2, max(ks), 128
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=12, m=min(64, n))
    Q, K, V = dev(w.Q * np.float32(gain), dtype), dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(13))
    idx = np.zeros((2, n), dtype=np.int32)
    for u in range(2):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV)
    pools = [torch.full(((Hkv * cap + 2 * guard) * d,), float("nan"), dtype=K.dtype, device=DEV) for _ in range(2)]
    Kc, Vc = (p[guard * d:guard * d + Hkv * cap * d].view(Hkv, cap, d) for p in pools)
    z.zipvl_compact_kv(K, V, idx_d, k_d, cap, Kc=Kc, Vc=Vc)
    O1, O2 = torch.zeros_like(Q), torch.zeros_like(Q)
    z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale, O=O1)
    z.zipvl_sparse_prefill(Q, Kc.view(B, Hkv, cap, d), Vc.view(B, Hkv, cap, d), idx_d, k_d, w.scale, z.KV_ALREADY_COMPACT, O=O2)
    torch.cuda.synchronize()
    assert torch.equal(O1, O2) and not torch.isnan(O2.float()).any()


@pytest.mark.parametrize("n,gain", [(400, 1.0), (448, 1.0), (448, 40.0)])
def test_attention_on_already_compacted_cache(n, gain):
    # the evicted cache is read in place, for n a multiple of the 64-row tile and not;
    # gain 40: logits far outside the range the offset-free pass accepts, so every workgroup repeats its keys
    say(f"attention KV_ALREADY_COMPACT n={n} gain={gain}")
    B, Hq, Hkv, d, dtype = 1, 4, 2, 128, "bf16"
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=8)
    if gain != 1.0:
        w.Q = torch.from_numpy(w.Q * np.float32(gain)).bfloat16().float().numpy()
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    ks = [211, 77]
    r = np.random.Generator(np.random.PCG64(9))
    idx = np.zeros((2, n), dtype=np.int32)
    for u in range(2):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV)
    Kc = torch.full((2, n, d), float("nan"), dtype=torch.bfloat16, device=DEV)   # rows beyond k stay NaN
    Vc = torch.full((2, n, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    z.zipvl_compact_kv(K, V, idx_d, k_d, n, Kc=Kc, Vc=Vc)
    O1 = z.zipvl_sparse_prefill(Q, K, V, idx_d, k_d, w.scale)
    O2 = z.zipvl_sparse_prefill(Q, Kc.view(B, Hkv, n, d), Vc.view(B, Hkv, n, d), idx_d, k_d, w.scale,
                                z.KV_ALREADY_COMPACT)
    torch.cuda.synchronize()
    assert not torch.isnan(O2.float()).any()
    assert torch.equal(O1, O2)
    Oh, G = host64(O2), Hq // Hkv
    worst = max(np.abs(Oh[0, h] - oz.kept_token_attention(w.Q[0, h], w.K[0, h // G], w.V[0, h // G], idx[h // G, :ks[h // G]], w.scale)).max()
                for h in range(Hq))
    say(f"  worst |dO| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


# ------------------------------------------------------------------ whole layer
def _edge_rows(p, r, extra):
    """Kept-token rows at the edges of the attention kernel's tiling (128 queries per workgroup, 32 per
    wave, 64 keys per tile): first and last rows of the first, a middle and the last query tile, rows on
    both sides of 64-key tile edges, the last kept row, plus `extra` random rows."""
    last_q, last_k, mid = (p - 1) // 128 * 128, (p - 1) // 64 * 64, (p // 2) // 128 * 128
    cand = [0, 1, 31, 32, 63, 64, 65, 127, 128, 129, mid - 1, mid, mid + 63, mid + 64, mid + 127,
            last_q - 1, last_q, last_k - 1, last_k, p - 2, p - 1]
    cand = [c for c in cand if 0 <= c < p]
    return np.unique(np.concatenate([np.array(cand, dtype=np.int64), r.integers(0, p, extra)]))


def _layer_parity(w, tau, sample_rows=None, heads=None, whole_heads=()):
    """Score, select, compaction and attention of one layer against the oracle.  The attention is run
    twice: on the original K, V (the library gathers K[T], V[T] itself), and exactly as the benchmark's
    step runs it - K and V read in place from the evicted cache (rows past k hold NaN), full-size output
    with the dropped rows cleared by the kernel.  Both outputs meet the oracle on every checked row.
    sample_rows=None: every row of the heads in `heads` (all heads when None).  Otherwise the tile-edge
    rows plus `sample_rows` random ones of those heads, and every row of the heads in `whole_heads`."""
    spec = w.spec
    B, Hq, Hkv, n, d, dtype = w.Q.shape[0], spec.Hq, spec.Hkv, spec.n, spec.d, spec.dtype
    G = Hq // Hkv
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    idx, k = z.zipvl_select(mass, rank, tau)
    Kc = torch.full((B * Hkv, n, d), float("nan"), dtype=Q.dtype, device=DEV)
    Vc = torch.full((B * Hkv, n, d), float("nan"), dtype=Q.dtype, device=DEV)
    _, _, ln = z.zipvl_compact_kv(K, V, idx, k, n, Kc=Kc, Vc=Vc)
    outs = {"gathered by the library": z.zipvl_sparse_prefill(Q, K, V, idx, k, w.scale)}
    O2 = torch.full((B, Hq, n, d), 7.0, dtype=Q.dtype, device=DEV)      # poison: every row must be rewritten
    z.zipvl_sparse_prefill(Q, Kc.view(B, Hkv, n, d), Vc.view(B, Hkv, n, d), idx, k, w.scale,
                           z.OUT_FULL | z.KV_ALREADY_COMPACT, O=O2)
    outs["evicted cache read in place (the benchmark's step)"] = O2
    torch.cuda.synchronize()
    mass_h, rank_h = mass.cpu().numpy(), rank.cpu().numpy()
    idx_h, k_h = idx.cpu().numpy(), k.cpu().numpy()
    assert ln.cpu().tolist() == k_h.tolist()
    kept = []
    for b in range(B):
        mo, ro = oz.token_scores(w.Q[b], w.K[b], w.probe_pos, w.scale)
        assert_scores_close(mass_h.reshape(B, Hkv, n)[b].astype(np.float64), mo, dtype, "mass")
        assert_scores_close(rank_h.reshape(B, Hkv, n)[b].astype(np.float64), ro, dtype, "rank")
        for g in range(Hkv):
            u = b * Hkv + g
            p, T = oz.select(mass_h[u], rank_h[u], tau)             # oracle fed the GPU's fp32 scores
            assert k_h[u] == p and np.array_equal(idx_h[u, :p], T), f"unit {u}: selection differs"
            kept.append(p / n)
            ko, vo, _ = oz.compact_kv(w.K[b, g], w.V[b, g], T)
            assert Kc[u, :p].to(torch.float32).cpu().numpy().tobytes() == ko.tobytes()
            assert Vc[u, :p].to(torch.float32).cpu().numpy().tobytes() == vo.tobytes()
    worst = {name: 0.0 for name in outs}
    r = np.random.Generator(np.random.PCG64(77))
    checked_rows = 0
    for b in range(B):
        for h in (range(Hq) if heads is None else sorted(set(heads) | set(whole_heads))):
            g = h // G
            u = b * Hkv + g
            T = idx_h[u, :k_h[u]]
            whole = sample_rows is None or h in whole_heads
            if whole:
                ref = oz.kept_token_attention(w.Q[b, h], w.K[b, g], w.V[b, g], T, w.scale)
                checked_rows += len(T)
            else:
                rows = _edge_rows(len(T), r, sample_rows)
                ref = oz.kept_token_attention_rows(w.Q[b, h], w.K[b, g], w.V[b, g], T, rows, w.scale)
                dropped = np.setdiff1d(np.arange(n), T)
                checked_rows += len(rows)
            for name, O in outs.items():
                Oh = host64(O[b, h])
                assert not np.isnan(Oh).any(), f"{name}: NaN in head {h}"
                if whole:
                    worst[name] = max(worst[name], np.abs(Oh - ref).max())       # dropped rows: ref is 0 there
                else:
                    worst[name] = max(worst[name], np.abs(Oh[T[rows]] - ref).max())
                    assert not Oh[dropped].any(), f"{name}: dropped rows must be zero"
    say(f"  kept {100 * np.mean(kept):.1f}% (min {100 * min(kept):.1f}, max {100 * max(kept):.1f}); {checked_rows} kept rows checked; "
        + "; ".join(f"worst |dO| {name} = {v:.3e}" for name, v in worst.items()))
    for name, v in worst.items():
        assert v <= ATOL_OUT[dtype], name
    return kept


def test_layer_cfg1_full():
    say("layer cfg1 (fp32, n=576)")
    w = make_workload(1)
    _layer_parity(w, w.tau)


def test_layer_with_hybrid_probe_set():
    say("layer with 64 recent + 64 random probes (bf16, GQA 6/2, n=2000)")
    n = 2000
    w = make_custom(1, 6, 2, n, 128, "bf16", seed=21, probe_pos=hybrid_probes(n, seed=5))
    assert len(w.probe_pos) == 128
    _layer_parity(w, 0.975)


# ------------------------------------------------------------------ all-rows (exact) scores
@pytest.mark.parametrize("case", [dict(B=1, Hq=4, Hkv=2, n=333, d=128, dtype="bf16"),
                                  dict(B=2, Hq=2, Hkv=2, n=200, d=64, dtype="f32"),
                                  dict(B=1, Hq=14, Hkv=2, n=700, d=128, dtype="bf16"),
                                  dict(B=1, Hq=2, Hkv=1, n=129, d=128, dtype="f32"),
                                  dict(B=1, Hq=2, Hkv=2, n=64, d=64, dtype="bf16"),
                                  dict(B=1, Hq=1, Hkv=1, n=1, d=128, dtype="bf16")])
def test_all_rows_scores_match_the_oracle(case):
    B, Hq, Hkv, n, d, dtype = (case[key] for key in ("B", "Hq", "Hkv", "n", "d", "dtype"))
    say(f"score_all_rows B={B} Hq={Hq} Hkv={Hkv} n={n} d={d} {dtype}")
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=71, m=min(64, n))
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    mass, rank = z.zipvl_score_all_rows(Q, K, w.scale)
    mass_only, none = z.zipvl_score_all_rows(Q, K, w.scale, want_rank=False)
    torch.cuda.synchronize()
    assert none is None and torch.equal(mass, mass_only)
    mass_h, rank_h = mass.cpu().numpy().astype(np.float64), rank.cpu().numpy().astype(np.float64)
    for b in range(B):
        mo, ro = oz.token_scores(w.Q[b], w.K[b], np.arange(n), w.scale)       # every row is a probe
        assert_scores_close(mass_h.reshape(B, Hkv, n)[b], mo, dtype, "mass")
        assert_scores_close(rank_h.reshape(B, Hkv, n)[b], ro, dtype, "rank")
    assert np.all(np.abs(mass_h.sum(axis=1) - 1.0) < 1e-4)


@pytest.mark.parametrize("n,d,dtype,gain", [(700, 128, "bf16", 12.0), (700, 128, "bf16", 80.0), (257, 64, "f32", 60.0), (129, 128, "f32", 12.0)])
def test_all_rows_scores_with_logits_that_outgrow_the_first_block(n, d, dtype, gain):
    """Logits far above those of the first keys, ragged lengths, strided inputs ([n, heads, d] in memory).
    A log2-domain exponent x carries sqrt(d) 2^-24 |x| < 1e-6 |x| from the fp32 product sum and its roundings."""
    say(f"score_all_rows n={n} d={d} {dtype} gain={gain}")
    w = make_custom(1, 4, 2, n, d, dtype, seed=72, m=64)
    K32 = w.K.copy()
    late = [n // 2, n - 30, n - 2]
    K32[:, :, late] = (gain / 4) * w.Q[:, ::2, late] / np.linalg.norm(w.Q[:, ::2, late], axis=-1, keepdims=True)
    Q = dev(w.Q, dtype).transpose(1, 2).contiguous().transpose(1, 2)
    K = dev(K32, dtype).transpose(1, 2).contiguous().transpose(1, 2)
    mass, rank = z.zipvl_score_all_rows(Q, K, w.scale)
    torch.cuda.synchronize()
    Qh, Kh = host64(Q)[0], host64(K)[0]
    big = max(np.abs(Qh[h] @ Kh[h // 2].T).max() for h in range(4)) * w.scale * 1.4427
    say(f"  largest log2-domain logit {big:.0f}")
    mo, ro = oz.token_scores(Qh, Kh, np.arange(n), w.scale)
    for got, ref in ((mass, mo), (rank, ro)):
        assert (np.abs(host64(got) - ref) <= 1e-9 + (1e-5 + 1e-6 * big) * np.abs(ref)).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_all_rows_scores_of_rows_32_mib_apart(dtype, d):
    """64 streamed rows that span 2 GiB and more are addressed with 64 bits per lane; bit for bit the contiguous result."""
    say(f"score_all_rows strides above 32 MiB {dtype} d={d}")
    n = 65
    w = make_custom(1, 1, 1, n, d, dtype, seed=74, m=64)
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    stride = (32 << 20) // K.element_size() + 64
    pool = torch.empty((n * stride,), dtype=K.dtype, device=DEV)
    Qs, Ks = (pool.as_strided((1, 1, n, d), (0, 0, stride, 1), off) for off in (0, d))
    Qs.copy_(Q)
    Ks.copy_(K)
    for a, b in zip(z.zipvl_score_all_rows(Q, K, w.scale), z.zipvl_score_all_rows(Qs, Ks, w.scale)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_all_rows_scores_keep_a_row_without_numbers_to_the_keys_it_sees(dtype, d, bad):
    """A query row that is not finite has no softmax; the scores of later keys, which it does not see, are those without it."""
    say(f"score_all_rows with a {bad} row {dtype} d={d}")
    n, rows = 203, (70, 192)                                 # inside a 32-row block; the first row of the last chunk
    w = make_custom(1, 4, 2, n, d, dtype, seed=73, m=64)
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    mass, rank = z.zipvl_score_all_rows(Q, K, w.scale)
    for i in rows:
        Qb = Q.clone()
        Qb[0, 3, i, 5] = bad                                 # query head 3 = unit 1
        mass_b, rank_b = z.zipvl_score_all_rows(Qb, K, w.scale)
        torch.cuda.synchronize()
        for a, b in ((mass, mass_b), (rank, rank_b)):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1, i + 1:], b[1, i + 1:])
            assert torch.isnan(b[1, :i + 1]).any()


def test_all_rows_scores_at_cfg2_shape_against_sampled_columns():
    say("score_all_rows at n=3072, 32 heads (sampled heads)")
    w = make_workload(2)
    spec = w.spec
    Q, K = dev(w.Q, spec.dtype), dev(w.K, spec.dtype)
    mass, rank = z.zipvl_score_all_rows(Q, K, w.scale)
    torch.cuda.synchronize()
    n = spec.n
    for u in (0, 13, 31):
        mo, ro = oz.token_scores(w.Q[0, u:u + 1], w.K[0, u:u + 1], np.arange(n), w.scale)
        assert_scores_close(mass[u].cpu().numpy().astype(np.float64)[None], mo, spec.dtype, "mass")
        assert_scores_close(rank[u].cpu().numpy().astype(np.float64)[None], ro, spec.dtype, "rank")


@pytest.mark.parametrize("B,Hq,Hkv,n,d,dtype", [(4, 26, 26, 2560, 128, "bf16"), (4, 28, 4, 2561, 64, "bf16"), (4, 28, 4, 2559, 128, "bf16"),
                                                (2, 20, 4, 2051, 128, "bf16"), (1, 16, 4, 2049, 64, "f32"), (1, 41, 41, 2048, 128, "bf16")])
def test_all_rows_scores_of_many_blocks(B, Hq, Hkv, n, d, dtype):
    """32 and 64 rows a wave on both sides of the line between them, blocks dealt in turned rounds and not, against a softmax in float64."""
    say(f"score_all_rows B={B} Hq={Hq} Hkv={Hkv} n={n} d={d} {dtype}")
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=75, m=64)
    Q, K = dev(w.Q, dtype), dev(w.K, dtype)
    mass, rank = z.zipvl_score_all_rows(Q, K, w.scale)
    G = Hq // Hkv
    hidden = torch.ones((n, n), dtype=torch.bool, device=DEV).triu(1)
    for b, g in {(0, 0), (B - 1, Hkv - 1), (0, Hkv // 2)}:
        a = torch.zeros((n,), dtype=torch.float64, device=DEV)
        for h in range(g * G, (g + 1) * G):
            logits = Q[b, h].double() @ K[b, g].double().t().contiguous() * w.scale
            a += torch.softmax(logits.masked_fill_(hidden, -math.inf), dim=1).sum(dim=0)
        a /= G
        u = b * Hkv + g
        assert_scores_close(host64(mass[u]), (a / n).cpu().numpy(), dtype, "mass")
        assert_scores_close(host64(rank[u]), (a / torch.arange(n, 0, -1, device=DEV)).cpu().numpy(), dtype, "rank")


# ------------------------------------------------------------------ one T per layer
def test_share_scores_bit_exact():
    say("share_scores")
    r = np.random.Generator(np.random.PCG64(41))
    for B, Hkv, n in ((1, 4, 18432), (3, 7, 1001), (2, 1, 77)):
        mass = r.random((B * Hkv, n)).astype(np.float32)
        mass /= mass.sum(axis=1, keepdims=True)
        rank = (mass * r.random((B * Hkv, n))).astype(np.float32)
        mb, rb = z.zipvl_share_scores(torch.from_numpy(mass).to(DEV), torch.from_numpy(rank).to(DEV), B)
        mb2, none = z.zipvl_share_scores(torch.from_numpy(mass).to(DEV), None, B)
        torch.cuda.synchronize()
        assert none is None
        for b in range(B):
            ref_m = oz.share_scores(mass[b * Hkv:(b + 1) * Hkv])
            assert mb[b].cpu().numpy().tobytes() == ref_m.tobytes()
            assert mb2[b].cpu().numpy().tobytes() == ref_m.tobytes()
            assert rb[b].cpu().numpy().tobytes() == oz.share_scores(rank[b * Hkv:(b + 1) * Hkv]).tobytes()


@pytest.mark.parametrize("case", [dict(B=2, Hq=8, Hkv=4, n=700, d=128, dtype="bf16", seed=51, full=True),
                                  dict(B=1, Hq=4, Hkv=4, n=333, d=64, dtype="f32", seed=52, full=True),
                                  dict(B=1, Hq=28, Hkv=4, n=4608, d=128, dtype="bf16", seed=53, full=False)])
def test_layer_with_one_important_set_per_batch_element(case):
    B, Hq, Hkv, n, d, dtype = (case[key] for key in ("B", "Hq", "Hkv", "n", "d", "dtype"))
    say(f"layer, one T per batch element: B={B} Hq={Hq} Hkv={Hkv} n={n} d={d} {dtype}")
    G, tau = Hq // Hkv, 0.975
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=case["seed"])
    Q, K, V = dev(w.Q, dtype), dev(w.K, dtype), dev(w.V, dtype)
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    mass_b, rank_b = z.zipvl_share_scores(mass, rank, B)
    idx, k = z.zipvl_select(mass_b, rank_b, tau)
    assert idx.shape == (B, n) and k.shape == (B,)
    Kc, Vc, ln = z.zipvl_compact_kv(K, V, idx, k, n, z.T_PER_BATCH)
    O = z.zipvl_sparse_prefill(Q, K, V, idx, k, w.scale, z.T_PER_BATCH)
    # the same attention from the evicted cache, compact output rows (every case: in-place K read and repack)
    Oc = z.zipvl_sparse_prefill(Q, Kc.view(B, Hkv, n, d), Vc.view(B, Hkv, n, d), idx, k, w.scale,
                                z.T_PER_BATCH | z.KV_ALREADY_COMPACT | z.OUT_COMPACT)
    torch.cuda.synchronize()
    mass_h, rank_h = mass.cpu().numpy(), rank.cpu().numpy()
    idx_h, k_h, ln_h = idx.cpu().numpy(), k.cpu().numpy(), ln.cpu().numpy()
    r = np.random.Generator(np.random.PCG64(78))
    worst = 0.0
    for b in range(B):
        # oracle fed the GPU's per-unit fp32 scores: same mean, same selection, exactly
        p, T = oz.select(oz.share_scores(mass_h[b * Hkv:(b + 1) * Hkv]), oz.share_scores(rank_h[b * Hkv:(b + 1) * Hkv]), tau)
        assert k_h[b] == p and np.array_equal(idx_h[b, :p], T), f"batch element {b}: selection differs"
        dropped = np.setdiff1d(np.arange(n), T)
        for g in range(Hkv):
            u = b * Hkv + g
            assert ln_h[u] == p
            ko, vo, _ = oz.compact_kv(w.K[b, g], w.V[b, g], T)
            assert Kc[u, :p].to(torch.float32).cpu().numpy().tobytes() == ko.tobytes()
            assert Vc[u, :p].to(torch.float32).cpu().numpy().tobytes() == vo.tobytes()
        for h in range(Hq):
            g = h // G
            Oh = host64(O[b, h])
            assert not Oh[dropped].any(), "dropped rows must be zero"
            if case["full"]:
                ref = oz.kept_token_attention(w.Q[b, h], w.K[b, g], w.V[b, g], T, w.scale)
                worst = max(worst, np.abs(Oh - ref).max())
                if Oc is not None:
                    worst = max(worst, np.abs(host64(Oc[b, h])[:p] - ref[T]).max())
            else:
                rows = np.unique(np.concatenate([[0, p - 1, min(127, p - 1), min(128, p - 1)], r.integers(0, p, 6)]))
                ref = oz.kept_token_attention_rows(w.Q[b, h], w.K[b, g], w.V[b, g], T, rows, w.scale)
                worst = max(worst, np.abs(Oh[T[rows]] - ref).max())
                worst = max(worst, np.abs(host64(Oc[b, h])[rows] - ref).max())
    say(f"  kept {[int(x) for x in k_h]} of {n}; worst |dO| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


# ------------------------------------------------------------------ mixed-precision cache
def _unpack(codes: np.ndarray, bits: int) -> np.ndarray:
    """[rows, d*bits/8] bytes -> [rows, d] codes (element c in bits [c*bits, c*bits+bits) of the row's bit string)."""
    per = 8 // bits
    out = np.empty((codes.shape[0], codes.shape[1] * per), dtype=np.uint8)
    for e in range(per):
        out[:, e::per] = (codes >> (bits * e)) & ((1 << bits) - 1)
    return out


def _check_qcache_against_oracle(cache, w, dtype, Ts, Hkv):
    """Codes and fp16 parameters of every unit, bit for bit; returns the oracle caches."""
    ref = []
    for u, T in enumerate(Ts):
        b, g = divmod(u, Hkv)
        qc = oz.quantize_kv(w.K[b, g], w.V[b, g], T)
        ref.append(qc)
        nh, nl = len(T), w.K.shape[2] - len(T)
        assert int(cache.len_hi[u]) == nh and int(cache.len_lo[u]) == nl
        for name, t in (("K", cache.K), ("V", cache.V)):
            for grp, bits, rows in (("hi", 4, nh), ("lo", 2, nl)):
                codes, scale, zero = qc[f"{name}_{grp}"]
                got = _unpack(t[f"{grp}_codes"][u, :rows].cpu().numpy(), bits)
                par = t[f"{grp}_params"][u, :rows].cpu().numpy()
                assert par[:, 0].tobytes() == scale.tobytes(), f"unit {u} {name} {grp}: scales differ"
                assert par[:, 1].tobytes() == zero.tobytes(), f"unit {u} {name} {grp}: zeros differ"
                bad = np.argwhere(got != codes)
                assert len(bad) == 0, f"unit {u} {name} {grp}: {len(bad)} codes differ, first at {bad[0]}"
    return ref


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 128), ("bf16", 64), ("f32", 64)])
def test_quantize_kv_bit_exact_and_decode_over_it(dtype, d):
    say(f"quantize_kv + decode_attn_q dtype={dtype} d={d}")
    B, Hq, Hkv, n = 2, 6, 3, 333
    G = Hq // Hkv
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=61)
    K, V = dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(62))
    ks = [1, 64, 333, 200, 17, 130]                           # k = n: the 2-bit group is empty
    idx = np.zeros((B * Hkv, n), dtype=np.int32)
    for u in range(B * Hkv):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    idx_d, k_d = torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV)
    cache = z.zipvl_quantize_kv(K, V, idx_d, k_d, n, n)
    torch.cuda.synchronize()
    ref = _check_qcache_against_oracle(cache, w, dtype, [idx[u, :ks[u]] for u in range(B * Hkv)], Hkv)

    # decode: one query per head over [4-bit rows | 2-bit rows | 3 appended rows]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    qh = r.standard_normal((B * Hq, d)).astype(np.float32)
    tail_k = r.standard_normal((3, B * Hkv, d)).astype(np.float32)
    tail_v = r.standard_normal((3, B * Hkv, d)).astype(np.float32)
    q = dev(qh, dtype)
    Kt = torch.zeros((B * Hkv, 8, d), dtype=tdt, device=DEV); Vt = torch.zeros_like(Kt)
    lt = torch.zeros((B * Hkv,), dtype=torch.int32, device=DEV)
    o0 = z.zipvl_decode_attn_q(q, cache, w.scale, B=B, Hq=Hq, Hkv=Hkv).float().cpu().numpy().astype(np.float64)
    for step in range(3):
        z.zipvl_kv_append(Kt, Vt, lt, dev(tail_k[step], dtype), dev(tail_v[step], dtype), B=B, Hkv=Hkv)
    o3 = z.zipvl_decode_attn_q(q, cache, w.scale, B=B, Hq=Hq, Hkv=Hkv, K_tail=Kt, V_tail=Vt, len_tail=lt)
    torch.cuda.synchronize()
    o3 = o3.float().cpu().numpy().astype(np.float64)
    q64 = host64(q)
    tk = host64(Kt)[:, :3]; tv = host64(Vt)[:, :3]
    worst = 0.0
    for bh in range(B * Hq):
        b, h = divmod(bh, Hq)
        u = b * Hkv + h // G
        worst = max(worst, np.abs(o0[bh] - oz.decode_attention_quantized(q64[bh], ref[u], w.scale)).max())
        worst = max(worst, np.abs(o3[bh] - oz.decode_attention_quantized(q64[bh], ref[u], w.scale, tk[u], tv[u])).max())
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 128), ("f32", 64), ("bf16", 64)])
def test_quantize_kv_codes_at_half_steps_and_degenerate_rows(dtype, d):
    """Quotients on and next to k + 1/2, constant rows, ranges whose fp16 scale is 0, subnormal or infinite: the codes are those
    of the correctly rounded division, bit for bit."""
    say(f"quantize_kv half steps dtype={dtype} d={d}")
    r = np.random.Generator(np.random.PCG64(63))
    n = 211
    X = np.empty((n, d), dtype=np.float32)
    for i in range(n):
        top = 15 if i % 2 else 3
        scale = np.float32(np.float16(2.0 ** r.integers(-12, 6) * (1 if i % 3 == 0 else r.uniform(1, 2))))
        zero = np.float32(np.float16(r.choice([0.0, -1.5, 3.25]) * scale))
        half = (r.integers(0, top, d) + 0.5).astype(np.float32)
        row = zero + scale * half
        row = np.where(r.random(d) < 0.3, np.nextafter(row, np.float32(r.choice([-1e9, 1e9]))), row)
        row[0], row[1] = zero, zero + scale * np.float32(top)
        X[i] = row
    X[5], X[6] = 0.75, 0.0                                    # constant rows: scale 0
    X[7] = r.standard_normal(d) * 1e6                         # scale and zero infinite in fp16
    X[8] = r.standard_normal(d) * 1e-9                        # scale rounds to 0
    X[9] = r.standard_normal(d) * 3e-7                        # subnormal scale
    X[10] = 3.0e4 * np.sign(r.standard_normal(d))             # finite zero, large scale
    K = dev(X, dtype).reshape(1, 1, n, d)
    idx = torch.zeros((1, n), dtype=torch.int32, device=DEV)
    odd = np.arange(1, n, 2)
    idx[0, :len(odd)] = torch.from_numpy(odd.astype(np.int32)).to(DEV)
    cache = z.zipvl_quantize_kv(K, K, idx, torch.tensor([len(odd)], dtype=torch.int32, device=DEV), n, n)
    torch.cuda.synchronize()
    Xh = host64(K)[0, 0].astype(np.float32)
    for t in (cache.K, cache.V):
        for name, bits, rows in (("hi", 4, odd), ("lo", 2, np.arange(0, n, 2))):
            with np.errstate(all="ignore"):
                codes, scale, zero = oz.quantize_rows(Xh[rows], bits)
            got = t[name + "_codes"][0, :len(rows)].cpu().numpy()
            got = ((got[:, :, None] >> (np.arange(8 // bits) * bits)) & (2 ** bits - 1)).reshape(len(rows), d)
            par = t[name + "_params"][0, :len(rows)].cpu().numpy()
            assert par[:, 0].tobytes() == scale.tobytes() and par[:, 1].tobytes() == zero.tobytes()
            finite = np.isfinite(scale) & np.isfinite(zero)               # inf / inf: the oracle's cast of NaN is not defined
            assert np.array_equal(got[finite], codes[finite])


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (8, 2), (14, 2)])
def test_decode_over_quantised_cache_for_every_group_size(Hq, Hkv):
    say(f"decode_attn_q Hq={Hq} Hkv={Hkv}")
    B, n, d, dtype = 1, 700, 128, "bf16"
    G = Hq // Hkv
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=65)
    K, V = dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(66))
    ks = [r.integers(1, n) for _ in range(Hkv)]
    idx = np.zeros((Hkv, n), dtype=np.int32)
    for u in range(Hkv):
        idx[u, :ks[u]] = np.sort(r.choice(n, ks[u], replace=False))
    cache = z.zipvl_quantize_kv(K, V, torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV), n, n)
    q = dev(r.standard_normal((Hq, d)).astype(np.float32), dtype)
    o = z.zipvl_decode_attn_q(q, cache, w.scale, B=B, Hq=Hq, Hkv=Hkv)
    torch.cuda.synchronize()
    worst = 0.0
    for h in range(Hq):
        u = h // G
        qc = oz.quantize_kv(w.K[0, u], w.V[0, u], idx[u, :ks[u]])
        worst = max(worst, np.abs(host64(o[h]) - oz.decode_attention_quantized(host64(q[h]), qc, w.scale)).max())
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= 2e-2


@pytest.mark.parametrize("dtype,d,G", [("bf16", 128, 1), ("f32", 64, 1), ("bf16", 128, 7), ("bf16", 64, 2), ("f32", 128, 4), ("f32", 64, 8)])
def test_decode_over_quantised_cache_at_tile_edges(dtype, d, G):
    """Part lengths (4-bit, 2-bit, appended) on both sides of the 16-row tiles, each part empty once; NaN in the appended rows
    that do not exist yet.  fp32: the oracle's dequantised rows are exact, the sums are not: 5e-5 of outputs of order one."""
    say(f"decode_attn_q tile edges dtype={dtype} d={d} G={G}")
    n, cap_t = 530, 40
    kept = [0, 1, 15, 16, 17, 33, 256, 514, 529, 530]
    tail = [0, 1, 15, 16, 17, 40, 0, 33, 1, 0]
    units = len(kept)
    w = make_custom(1, units * G, units, n, d, dtype, seed=67)
    r = np.random.Generator(np.random.PCG64(68))
    idx = np.zeros((units, n), dtype=np.int32)
    for u, k in enumerate(kept):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    cache = z.zipvl_quantize_kv(dev(w.K, dtype), dev(w.V, dtype), torch.from_numpy(idx).to(DEV),
                                torch.tensor(kept, dtype=torch.int32, device=DEV), n, n)
    q = dev(r.standard_normal((units * G, d)).astype(np.float32), dtype)
    Kt, Vt = (dev(r.standard_normal((units, cap_t, d)).astype(np.float32), dtype) for _ in range(2))
    for u, t in enumerate(tail):
        Kt[u, t:] = float("nan")
        Vt[u, t:] = float("nan")
    o = z.zipvl_decode_attn_q(q, cache, w.scale, B=1, Hq=units * G, Hkv=units, K_tail=Kt, V_tail=Vt,
                              len_tail=torch.tensor(tail, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    worst = 0.0
    for u, (k, t) in enumerate(zip(kept, tail)):
        qc = oz.quantize_kv(w.K[0, u], w.V[0, u], idx[u, :k])
        for h in range(u * G, u * G + G):
            ref = oz.decode_attention_quantized(host64(q[h]), qc, w.scale, host64(Kt[u, :t]), host64(Vt[u, :t]))
            worst = max(worst, np.abs(host64(o[h]) - ref).max())
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= (2e-2 if dtype == "bf16" else 5e-5)


@pytest.mark.parametrize("Hq,Hkv,n,fine", [(14, 2, 6300, 50), (28, 4, 6104, 24), (28, 4, 6105, 49), (18, 2, 9000, 64), (32, 8, 6300, 32)])
def test_decode_of_groups_over_quantised_caches_splits_by_what_the_workspace_holds(Hq, Hkv, n, fine):
    """Groups of bf16 at d = 128 have splits of 128 rows over long quantised caches too (from 25 splits of 256 on, at most 256 workgroups): a workspace of the size asked
    for and the smallest one, with a full and a nearly empty unit, against the oracle; nothing is written past the end of either, and a byte less is refused."""
    say(f"decode_attn_q groups {Hq}/{Hkv} n={n}")
    d, G, k, cap_t, tail = 128, Hq // Hkv, 2000, 40, 33
    cap = n + cap_t
    w = make_custom(1, Hq, Hkv, n, d, "bf16", seed=87)
    r = np.random.Generator(np.random.PCG64(88))
    idx = np.zeros((Hkv, n), dtype=np.int32)
    for u in range(Hkv):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    cache = z.zipvl_quantize_kv(dev(w.K, "bf16"), dev(w.V, "bf16"), torch.from_numpy(idx).to(DEV), torch.full((Hkv,), k, dtype=torch.int32, device=DEV), k, n - k)
    cache.len_hi[1], cache.len_lo[1] = 20, 33
    q = dev(r.standard_normal((Hq, d)).astype(np.float32), "bf16")
    Kt, Vt = (dev(r.standard_normal((Hkv, cap_t, d)).astype(np.float32), "bf16") for _ in range(2))
    lt = torch.full((Hkv,), tail, dtype=torch.int32, device=DEV)
    state = Hq * (d + 2) * 4
    least = -(-cap // 256) * state
    full = z.workspace_bytes(z.OP_DECODE_Q, z.dims_of(None, None, None, B=1, Hq=Hq, Hkv=Hkv, n=cap, d=d, dtype=1))
    assert full == fine * state
    args = dict(B=1, Hq=Hq, Hkv=Hkv, K_tail=Kt, V_tail=Vt, len_tail=lt)
    for size in sorted({full, least}):
        room = torch.full((size + 256,), 0xA5, dtype=torch.uint8, device=DEV)
        o = z.zipvl_decode_attn_q(q, cache, w.scale, ws=room[:size], o=torch.empty_like(q), **args)
        torch.cuda.synchronize()
        assert bool((room[size:] == 0xA5).all())
        for u in (0, 1, Hkv - 1):
            qc = oz.quantize_kv(w.K[0, u], w.V[0, u], idx[u, :k])
            if u == 1:
                qc = {name: tuple(x[:rows] for x in qc[name]) for name, rows in (("K_hi", 20), ("K_lo", 33), ("V_hi", 20), ("V_lo", 33))}
            for h in (u * G, u * G + G - 1):
                ref = oz.decode_attention_quantized(host64(q[h]), qc, w.scale, host64(Kt[u, :tail]), host64(Vt[u, :tail]))
                assert np.abs(host64(o[h]) - ref).max() <= ATOL_OUT["bf16"], f"{size} bytes, head {h}"
    with pytest.raises(z.ZipvlError):
        z.zipvl_decode_attn_q(q, cache, w.scale, ws=room[:least - 1], o=torch.empty_like(q), **args)


def _one_head_cache(K, V, kept, copies):
    """The mixed-precision cache of a few heads K, V [heads, n, d], `copies` times over: with 300 units and more a launch
    splits a unit's rows two or three ways, so that every wave takes several blocks of 64 rows of either part."""
    heads, n, d = K.shape
    r = np.random.Generator(np.random.PCG64(n + d))
    idx = np.zeros((heads, n), dtype=np.int32)
    for h in range(heads):
        idx[h, :kept] = np.sort(r.choice(n, kept, replace=False))
    grow = lambda x: dev(x, "f32")[None].expand(copies, -1, -1, -1)
    cache = z.zipvl_quantize_kv(grow(K), grow(V), torch.from_numpy(idx).to(DEV).repeat(copies, 1),
                                torch.full((copies * heads,), kept, dtype=torch.int32, device=DEV), kept, n - kept)
    return cache, idx


def _check_one_head(name, q, K, V, kept, bound, copies=110):
    """|do| of every channel against `bound` times what the channel's rows weigh in all, sum_j p_j |v_j| (float64, from the codes)."""
    heads, n, d = K.shape
    scale = 1.0 / math.sqrt(d)
    cache, idx = _one_head_cache(K, V, kept, copies)
    o = z.zipvl_decode_attn_q(dev(np.tile(q, (copies, 1)), "f32"), cache, scale, B=copies, Hq=heads, Hkv=heads)
    torch.cuda.synchronize()
    assert torch.equal(o, o[:heads].repeat(copies, 1))       # every copy the same bits
    worst = 0.0
    for h in range(heads):
        qc = oz.quantize_kv(K[h], V[h], idx[h, :kept])
        ref = oz.decode_attention_quantized(q[h].astype(np.float64), qc, scale)
        s = np.concatenate([oz.dequantize_rows(*qc["K_hi"]), oz.dequantize_rows(*qc["K_lo"])]) @ q[h].astype(np.float64) * scale
        p = np.exp(s - s.max())
        v = np.concatenate([oz.dequantize_rows(*qc["V_hi"]), oz.dequantize_rows(*qc["V_lo"])])
        worst = max(worst, float((np.abs(host64(o[h]) - ref) / (p @ np.abs(v) / p.sum())).max()))
    say(f"  {name}: worst |do| / sum p |v| = {worst:.2e} (bound {bound:.1e})")
    assert worst <= bound, f"{name}: {worst:.3e}"


@pytest.mark.parametrize("d", [64, 128])
def test_one_head_decode_over_quantised_cache_keeps_its_precision_as_the_offset_moves(d):
    """Rows of V that get smaller by seven orders of magnitude while the logits rise by 60, and large rows that later ones
    outweigh: whatever was summed before, the rows that count are weighed in full.  Bound: log2-domain scores up to s = 90 in
    fp32, two roundings of each and one of their sum: 3 * 2^-24 * 90 * ln 2 = 1.1e-5 of a weight, 2 to 3 times that with the
    query's and the exponential's: 3e-5."""
    say(f"decode_attn_q one head, offset and scale move, d={d}")
    n, heads = 4000, 3
    r = np.random.Generator(np.random.PCG64(81))
    q = (r.standard_normal((heads, d)) + 1).astype(np.float32)
    K, V = (r.standard_normal((heads, n, d)).astype(np.float32) for _ in range(2))
    at = np.arange(n) / n
    rise = np.stack([60 * at, 35 * (at > 0.7), 40 * (at * 8 % 1)])                   # logits of the three heads along the sequence
    size = np.stack([10.0 ** (4 - 7 * at), np.where(at > 0.7, 1e-3, 1e4), np.where(at * 8 % 1 > 0.8, 1e-2, 1e3)])
    unit = q / (q * q).sum(1, keepdims=True) * math.sqrt(d)                          # adds one to a head's logits
    K += (rise[:, :, None] * unit[:, None, :]).astype(np.float32)
    V *= size[:, :, None].astype(np.float32)
    for kept in (1000, 4000 - 64, 64):
        _check_one_head(f"kept {kept}", q, K, V, kept, 3e-5)


@pytest.mark.parametrize("d", [64, 128])
def test_one_head_decode_over_quantised_cache_with_outliers_in_v(d):
    """One channel of V far above or far below the others, which then share the lowest or the highest code of their rows, and
    rows that are nearly constant: every channel to fp32 accuracy, not only the large one.  Bound: log2-domain scores up to
    s = 12 in fp32, three roundings, 3 * 2^-24 * 12 * ln 2 = 1.5e-6 of a weight, and 2^-23 of its exponential: 2e-6."""
    say(f"decode_attn_q one head, outliers in V, d={d}")
    n, heads = 4000, 4
    r = np.random.Generator(np.random.PCG64(83))
    q = (r.standard_normal((heads, d)) + 1).astype(np.float32)
    K, V = (r.standard_normal((heads, n, d)).astype(np.float32) for _ in range(2))
    V[0, :, 7] += 1000
    V[1, :, 9] -= 1000
    V[2, ::3] = 100 + 1e-2 * V[2, ::3]
    for kept in (1000, 4000 - 64):
        _check_one_head(f"kept {kept}", q, K, V, kept, 2e-6)


@pytest.mark.parametrize("d", [64, 128])
def test_one_head_decode_over_quantised_cache_with_outliers_in_k(d):
    """One channel of K far above or far below the others, which the query hardly looks at, and one of the query where all K are
    0: the scores are the small sum of large terms.  Bound: log2-domain scores up to s = 128 in fp32, a rounding of each and one
    of the difference to the largest: 2 * 2^-24 * 128 * ln 2 = 1.1e-5 of a weight, as much for its exponential: 2.2e-5."""
    say(f"decode_attn_q one head, outliers in K, d={d}")
    n, heads = 4000, 4
    r = np.random.Generator(np.random.PCG64(85))
    q = (r.standard_normal((heads, d)) + 1).astype(np.float32)
    K, V = (r.standard_normal((heads, n, d)).astype(np.float32) for _ in range(2))
    K[0, :, 7] += 1000
    K[1, :, 9] -= 1000
    q[0, 7] = q[1, 9] = 1e-3
    K[2] = np.abs(K[2])
    K[2, :, 11] = 0
    q[2, 11] = 1000
    for kept in (1000, 4000 - 64):
        _check_one_head(f"kept {kept}", q, K, V, kept, 2.2e-5)


@pytest.mark.parametrize("d", [64, 128])
def test_one_head_decode_over_quantised_cache_in_blocks_of_64_rows(d):
    """Integer products: both parts around multiples of 64 rows, in few units (a wave takes one block of either part; several
    blocks, whose scale and offset move: above); value rows from 1e-4 to 1e4; logits that rise along the sequence; query elements
    six orders of magnitude apart, and a query of zeros.  Bound: a score of |s| is off by up to 4 * 2^-24 |s| in fp32, a
    weight by that relative amount; |s| < 80 here, so 2e-5 of the largest value of the head."""
    say(f"decode_attn_q one head, blocks of 64, d={d}")
    n = 400
    kept = [0, 1, 63, 64, 65, 127, 128, 129, 192, 336, 399, 400]
    units = len(kept)
    r = np.random.Generator(np.random.PCG64(71))
    w = make_custom(1, units, units, n, d, "f32", seed=72)
    q = r.standard_normal((units, d)).astype(np.float32)
    q[1] *= np.float32(10.0) ** r.uniform(-6, 0, d).astype(np.float32)
    q[2] = 0
    mag = np.concatenate([np.full(100, 1e-4), 10.0 ** r.uniform(-4, 4, 200), np.full(100, 1e-4)]).astype(np.float32)
    V = (w.V * mag[None, None, :, None]).astype(np.float32)
    K = (w.K + 0.06 * np.arange(n, dtype=np.float32)[None, None, :, None] * q[None, :, None, :] / np.maximum(np.linalg.norm(q, axis=1), 1e-3)[None, :, None, None]).astype(np.float32)
    idx = np.zeros((units, n), dtype=np.int32)
    for u, k in enumerate(kept):
        idx[u, :k] = np.sort(r.choice(n, k, replace=False))
    cache = z.zipvl_quantize_kv(dev(K, "f32"), dev(V, "f32"), torch.from_numpy(idx).to(DEV), torch.tensor(kept, dtype=torch.int32, device=DEV), n, n)
    o = z.zipvl_decode_attn_q(dev(q, "f32"), cache, w.scale, B=1, Hq=units, Hkv=units)
    torch.cuda.synchronize()
    for u, k in enumerate(kept):
        qc = oz.quantize_kv(K[0, u], V[0, u], idx[u, :k])
        ref = oz.decode_attention_quantized(q[u].astype(np.float64), qc, w.scale)
        err = np.abs(host64(o[u]) - ref).max()
        assert err <= 2e-5 * np.abs(V[0, u]).max(), f"unit {u}: {err:.3e}"


def test_quantize_kv_with_one_set_per_batch_element_and_without_T():
    say("quantize_kv T_PER_BATCH / idx=NULL")
    B, Hq, Hkv, n, d, dtype = 2, 4, 4, 1000, 128, "bf16"
    w = make_custom(B, Hq, Hkv, n, d, dtype, seed=63)
    K, V = dev(w.K, dtype), dev(w.V, dtype)
    r = np.random.Generator(np.random.PCG64(64))
    ks = [411, 77]
    idx = np.zeros((B, n), dtype=np.int32)
    for b in range(B):
        idx[b, :ks[b]] = np.sort(r.choice(n, ks[b], replace=False))
    cache = z.zipvl_quantize_kv(K, V, torch.from_numpy(idx).to(DEV), torch.tensor(ks, dtype=torch.int32, device=DEV),
                                n, n, z.T_PER_BATCH)
    torch.cuda.synchronize()
    _check_qcache_against_oracle(cache, w, dtype, [idx[u // Hkv, :ks[u // Hkv]] for u in range(B * Hkv)], Hkv)
    allhi = z.zipvl_quantize_kv(K, V, None, None, n, 8)       # every token important
    torch.cuda.synchronize()
    _check_qcache_against_oracle(allhi, w, dtype, [np.arange(n)] * (B * Hkv), Hkv)


@pytest.mark.parametrize("n,k,shared", [(1, 1, False), (2, 1, False), (33, 32, True), (64, 20, False), (65, 64, False), (129, 1, False), (4160, 4097, True),
                                        (20001, 9000, False), (70001, 5000, True)])
def test_quantize_kv_takes_positions_in_any_order(n, k, shared):
    """T shuffled, and shuffled among positions that are none: the cache of T in ascending order, with a workspace of no more bytes than
    asked for; the ascending one against the oracle's ranks.  At both edges of a block of 64 tokens and of a word of 32, with more kept tokens
    than are taken at a time, and with more blocks than threads."""
    say(f"quantize_kv positions in any order n={n} k={k} shared={shared}")
    B, Hkv, d = 2, 2, 64
    r = np.random.Generator(np.random.PCG64(n))
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    K, V = (torch.randn((B, Hkv, n, d), generator=g, device=DEV) for _ in range(2))
    sets = B if shared else B * Hkv
    T = [np.sort(r.choice(n, max(1, k - s), replace=False)) for s in range(sets)]
    none = [-1, n, n + 70, -2**31, 2**31 - 1][:n - k]
    flag = z.T_PER_BATCH if shared else 0
    need = z.workspace_bytes(z.OP_QUANTIZE_KV, z.dims_of(None, K, V, Hq=Hkv))

    def cache(order):
        rows = [order(t) for t in T]
        idx = np.zeros((sets, n), dtype=np.int32)
        for s, t in enumerate(rows):
            idx[s, :len(t)] = t
        c = z.QCache(B * Hkv, n, n, d, DEV)
        for t in (c.K, c.V):
            for x in t.values():
                x.zero_()
        ws = torch.full((need + 64,), 0x5A, dtype=torch.uint8, device=DEV)
        z.zipvl_quantize_kv(K, V, torch.from_numpy(idx).to(DEV), torch.tensor([len(t) for t in rows], dtype=torch.int32, device=DEV), n, n, flag,
                            cache=c, ws=ws[:need])
        torch.cuda.synchronize()
        assert bool((ws[need:] == 0x5A).all())
        return c

    plain = cache(lambda t: t)
    for order in (lambda t: r.permutation(t), lambda t: r.permutation(np.concatenate([t, none]))):
        other = cache(order)
        for a, b in ((plain.K, other.K), (plain.V, other.V)):
            assert all(torch.equal(a[x].view(torch.uint8), b[x].view(torch.uint8)) for x in a)
    for u in (0, B * Hkv - 1):
        t = T[u // Hkv if shared else u]
        qc = oz.quantize_kv(K.view(B * Hkv, n, d)[u].cpu().numpy(), V.view(B * Hkv, n, d)[u].cpu().numpy(), t)
        for name, x in (("K", plain.K), ("V", plain.V)):
            for part, rows in (("hi", len(t)), ("lo", n - len(t))):
                scale, zero = qc[f"{name}_{part}"][1:]
                params = x[f"{part}_params"][u, :rows].cpu().numpy()
                assert np.array_equal(params[:, 0], scale) and np.array_equal(params[:, 1], zero)


def test_quantised_cache_at_stack_shape_sampled_units():
    say("quantize_kv + decode_attn_q at B4 H32 n8192 (sampled units)")
    from workloads import make_stack_layer_device
    Q, K, V, probe, scale = make_stack_layer_device(7, DEV)
    B, H, n, d = K.shape
    mass, rank = z.zipvl_score(Q, K, probe, scale)
    idx, k = z.zipvl_select(mass, rank, 0.975)
    cache = z.zipvl_quantize_kv(K, V, idx, k, n, n)
    g = torch.Generator(device=DEV); g.manual_seed(5)
    q = torch.randn((B * H, d), generator=g, device=DEV).to(torch.bfloat16)
    o = z.zipvl_decode_attn_q(q, cache, scale, B=B, Hq=H, Hkv=H)
    torch.cuda.synchronize()
    k_h, idx_h = k.cpu().numpy(), idx.cpu().numpy()
    assert cache.len_hi.cpu().tolist() == k_h.tolist() and cache.len_lo.cpu().tolist() == (n - k_h).tolist()
    worst = 0.0
    for u in (0, 37, 127):
        b, h = divmod(u, H)
        Kh, Vh = K[b, h].float().cpu().numpy(), V[b, h].float().cpu().numpy()
        qc = oz.quantize_kv(Kh, Vh, idx_h[u, :k_h[u]])
        for name, t in (("K", cache.K), ("V", cache.V)):
            assert np.array_equal(_unpack(t["hi_codes"][u, :k_h[u]].cpu().numpy(), 4), qc[name + "_hi"][0])
            assert np.array_equal(_unpack(t["lo_codes"][u, :n - k_h[u]].cpu().numpy(), 2), qc[name + "_lo"][0])
        refo = oz.decode_attention_quantized(host64(q[u]), qc, scale)
        worst = max(worst, np.abs(host64(o[u]) - refo).max())
    bits = 8.0 * cache.nbytes() / (2.0 * B * H * n * d)
    say(f"  kept {100 * k_h.mean() / n:.1f}% at 4 bits; {bits:.2f} bits per element incl. parameters "
        f"(compression {16 / bits:.2f}x at full capacity arrays); worst |do| = {worst:.3e}")
    assert worst <= 2e-2


def test_layer_tau_one_is_dense_attention():
    say("layer tau=1")
    w = make_custom(1, 4, 2, 320, 128, "bf16", seed=12)
    Q, K, V = dev(w.Q, "bf16"), dev(w.K, "bf16"), dev(w.V, "bf16")
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    idx, k = z.zipvl_select(mass, rank, 1.0)
    O = z.zipvl_sparse_prefill(Q, K, V, idx, k, w.scale)
    torch.cuda.synchronize()
    assert k.cpu().tolist() == [320, 320]
    for h in range(4):
        ref = oz.dense_causal_attention(w.Q[0, h], w.K[0, h // 2], w.V[0, h // 2], w.scale)
        assert np.abs(host64(O[0, h]) - ref).max() <= 2e-2


def test_layer_cfg2_sampled():
    say("layer cfg2 (bf16, 32 heads, n=3072), sampled output rows")
    w = make_workload(2)
    _layer_parity(w, w.tau, sample_rows=8, heads=range(32), whole_heads=[0, 13, 31])


def test_layer_cfg3_three_taus_selection_and_sampled_rows():
    say("layer cfg3 (bf16, 40 heads, n=4096)")
    w = make_workload(3)
    ks = []
    for tau in w.spec.taus:
        kept = _layer_parity(w, tau, sample_rows=4, heads=range(0, 40, 3), whole_heads=[7] if tau == w.tau else [])
        ks.append(np.mean(kept))
    assert ks[0] <= ks[1] <= ks[2]


def test_layer_cfg4_headline_shape_sampled():
    say("layer cfg4 (bf16 GQA 28/4, n=18432): one whole query head per KV group, tile-edge rows of all 28 heads")
    w = make_workload(4)
    _layer_parity(w, w.tau, sample_rows=6, heads=range(28), whole_heads=[0, 9, 18, 27])


def test_layer_beyond_the_benchmark_lengths_sampled():
    say("layer at n=40960 (bf16 GQA 2/1): selection keys no longer fit LDS, 320 query tiles per head")
    w = make_custom(1, 2, 1, 40960, 128, "bf16", seed=81, spike_frac=0.05)
    _layer_parity(w, 0.975, sample_rows=10)


def test_layer_cfg5_first_and_last_layer_then_decode_on_evicted_cache():
    say("layer cfg5 (bf16, 32 heads, n=8192), layers 0, 10, 21 and 31 of the ramp, batch slice of 1; then decode on the evicted cache")
    fracs = []
    for layer in (0, 10, 21, 31):
        w = make_workload(5, layer=layer, batch=1)
        kept = _layer_parity(w, w.tau, sample_rows=4, heads=[3, 17, 30], whole_heads=[30] if layer == 31 else [])
        fracs.append(np.mean(kept))
    assert max(fracs) - min(fracs) > 0.05          # the spike ramp makes the kept ratio layer dependent
    # decode: two steps against the evicted cache of the last layer
    spec = w.spec
    Q, K, V = dev(w.Q, "bf16"), dev(w.K, "bf16"), dev(w.V, "bf16")
    mass, rank = z.zipvl_score(Q, K, w.probe_pos, w.scale)
    idx, k = z.zipvl_select(mass, rank, w.tau)
    cap = int(k.max().item()) + 4
    Kc, Vc, ln = z.zipvl_compact_kv(K, V, idx, k, cap)
    r = np.random.Generator(np.random.PCG64(5))
    from workloads import round_to_bf16
    H, d = spec.Hq, spec.d
    idx_h, k_h = idx.cpu().numpy(), k.cpu().numpy()
    Kh = [w.K[0, g][idx_h[g, :k_h[g]]] for g in range(H)]
    Vh = [w.V[0, g][idx_h[g, :k_h[g]]] for g in range(H)]
    for step in range(2):
        q = round_to_bf16(r.standard_normal((H, d)).astype(np.float32))
        kn = round_to_bf16(r.standard_normal((H, d)).astype(np.float32))
        vn = round_to_bf16(r.standard_normal((H, d)).astype(np.float32))
        z.zipvl_kv_append(Kc, Vc, ln, dev(kn, "bf16"), dev(vn, "bf16"), B=1, Hkv=H)
        o = z.zipvl_decode_attn(dev(q, "bf16"), Kc, Vc, ln, w.scale, B=1, Hq=H, Hkv=H)
        torch.cuda.synchronize()
        oh = host64(o)
        for g in (0, 17, 31):
            ref, Kh[g], Vh[g], _ = oz.decode_step(q[g], kn[g], vn[g], Kh[g], Vh[g], len(Kh[g]), w.scale)
            assert np.abs(oh[g] - ref).max() <= 2e-2
        for g in range(H):
            if g not in (0, 17, 31):
                Kh[g] = np.concatenate([Kh[g], kn[g][None]]); Vh[g] = np.concatenate([Vh[g], vn[g][None]])
    assert ln.cpu().tolist() == [int(x) + 2 for x in k_h]


# ------------------------------------------------------------------ decode
@pytest.mark.parametrize("dtype,d,Hq,Hkv", [("bf16", 128, 4, 4), ("bf16", 128, 14, 2), ("f32", 64, 4, 2), ("bf16", 64, 3, 1)])
def test_decode_append_and_attention(dtype, d, Hq, Hkv):
    say(f"decode dtype={dtype} d={d} Hq={Hq} Hkv={Hkv}")
    B, cap = 2, 1300
    G = Hq // Hkv
    units = B * Hkv
    w = make_custom(B, Hq, Hkv, cap, d, dtype, seed=31)
    Kc = dev(w.K, dtype).reshape(units, cap, d).clone()
    Vc = dev(w.V, dtype).reshape(units, cap, d).clone()
    lens = [1, 1299, 640, 17][:units] + [5] * max(0, units - 4)
    ln = torch.tensor(lens, dtype=torch.int32, device=DEV)
    r = np.random.Generator(np.random.PCG64(32))
    from workloads import round_to_bf16
    cast = round_to_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    q = cast(r.standard_normal((B * Hq, d)).astype(np.float32) * 2)
    kn = cast(r.standard_normal((units, d)).astype(np.float32))
    vn = cast(r.standard_normal((units, d)).astype(np.float32))
    z.zipvl_kv_append(Kc, Vc, ln, dev(kn, dtype), dev(vn, dtype), B=B, Hkv=Hkv)
    o = z.zipvl_decode_attn(dev(q, dtype), Kc, Vc, ln, w.scale, B=B, Hq=Hq, Hkv=Hkv)
    torch.cuda.synchronize()
    assert ln.cpu().tolist() == [x + 1 for x in lens]
    oh = host64(o)
    Kh, Vh = w.K.reshape(units, cap, d), w.V.reshape(units, cap, d)
    worst = 0.0
    for b in range(B):
        for h in range(Hq):
            u = b * Hkv + h // G
            ref, Ko, Vo, L1 = oz.decode_step(q[b * Hq + h], kn[u], vn[u], Kh[u], Vh[u], lens[u], w.scale)
            worst = max(worst, np.abs(oh[b * Hq + h] - ref).max())
            assert Kc[u, lens[u]].to(torch.float32).cpu().numpy().tobytes() == kn[u].tobytes()
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


@pytest.mark.parametrize("dtype,d,B,Hq,Hkv", [("bf16", 128, 1, 28, 4), ("bf16", 128, 2, 4, 4), ("f32", 128, 1, 7, 1), ("f32", 64, 1, 4, 4), ("bf16", 64, 1, 8, 1),
                                              ("bf16", 128, 1, 18, 2), ("bf16", 128, 9, 7, 7)])
@pytest.mark.parametrize("cap", [1, 64, 65, 129, 1000, 6400])
def test_decode_splits_by_what_the_workspace_holds(dtype, d, B, Hq, Hkv, cap):
    """Splits of fewer rows where few heads leave the chip idle: a workspace of the size asked for, and the smallest one (splits of 256 rows), in both
    entry points, against the oracle; nothing is written past the end of either, and one byte less than the smallest is refused."""
    say(f"decode splits {dtype} d={d} {B}x{Hq}/{Hkv} cap={cap}")
    G, units = Hq // Hkv, B * Hkv
    w = make_custom(B, Hq, Hkv, cap, d, dtype, seed=33)
    Kc, Vc = (dev(x, dtype).reshape(units, cap, d) for x in (w.K, w.V))
    lens = [max(0, cap - 1 - 37 * u) for u in range(units)]
    r = np.random.Generator(np.random.PCG64(34))
    cast = (lambda x: torch.from_numpy(x).bfloat16().float().numpy()) if dtype == "bf16" else (lambda x: x)
    q, kn, vn = (cast(r.standard_normal((rows, d)).astype(np.float32)) for rows in (B * Hq, units, units))
    refs = [oz.decode_step(q[i], kn[i // G], vn[i // G], Kc[i // G].float().cpu().numpy(), Vc[i // G].float().cpu().numpy(), lens[i // G], w.scale)[0]
            for i in range(B * Hq)]
    dm = z.dims_of(None, None, None, B=B, Hq=Hq, Hkv=Hkv, n=cap, d=d, dtype=1 if dtype == "bf16" else 0)
    per = max(256, ((cap + 15) // 16 + 15) // 16 * 16)
    least = max(min(-(-1024 // units), -(-cap // 256)), -(-cap // per)) * B * Hq * (d + 2) * 4
    full, counters = z.workspace_bytes(z.OP_DECODE, dm), z.workspace_bytes(z.OP_DECODE_STEP, dm) - z.workspace_bytes(z.OP_DECODE, dm)
    assert full >= least
    for size in {full, least}:
        K1, V1, ln = Kc.clone(), Vc.clone(), torch.tensor(lens, dtype=torch.int32, device=DEV)
        room = torch.zeros(counters + size + 256, dtype=torch.uint8, device=DEV)
        room[counters + size:] = 0xA5
        args = dict(B=B, Hq=Hq, Hkv=Hkv)
        step = z.zipvl_decode_step(dev(q, dtype), K1, V1, ln, dev(kn, dtype), dev(vn, dtype), w.scale, ws=room[:counters + size], **args)
        assert ln.cpu().tolist() == [x + 1 for x in lens]
        attn = z.zipvl_decode_attn(dev(q, dtype), K1, V1, ln, w.scale, ws=room[counters:counters + size], **args)
        torch.cuda.synchronize()
        assert torch.equal(step, attn)
        assert bool((room[counters + size:] == 0xA5).all()) and not room[:counters].any()
        worst = max(np.abs(host64(step[i]) - refs[i]).max() for i in range(B * Hq))
        assert worst <= ATOL_OUT[dtype], f"{size} bytes: {worst:.3e}"
    with pytest.raises(z.ZipvlError):
        z.zipvl_decode_attn(dev(q, dtype), Kc, Vc, ln, w.scale, ws=room[counters:counters + least - 1], **args)


# units of one head, cap, splits of 256 rows, finer ones, tiles of 16 rows from which a unit has the finer ones
@pytest.mark.parametrize("dtype,d,units,cap,coarse,fine,first", [("bf16", 128, 8, 2700, 11, 22, 61), ("f32", 64, 8, 2700, 11, 22, 61), ("bf16", 64, 32, 1300, 6, 9, 41),
                                                                 ("bf16", 128, 4, 1300, 6, 11, 0), ("f32", 128, 4, 700, 3, 11, 0), ("bf16", 128, 64, 723, 3, 6, 14), ("bf16", 128, 32, 3461, 14, 16, 168), ("f32", 64, 56, 1015, 4, 7, 21), ("f32", 64, 16, 5500, 22, 22, 0)])
def test_decode_of_one_head_has_finer_splits_where_a_cache_is_full(dtype, d, units, cap, coarse, fine, first):
    """Splits finer than 256 rows pay in long caches only: a unit below the line leaves as many partial states as with the smallest workspace, one above it
    as many as there is room for, in one call; outputs against the oracle, and the fused step over the same rows gives the same bits."""
    say(f"finer splits {dtype} d={d} units={units} cap={cap}")
    tiles = lambda rows: -(-rows // 16)
    states = lambda rows: max(1, -(-tiles(rows) // max(1, -(-tiles(rows) // (coarse if tiles(rows) < first else fine)))))
    edge = 16 * first if first else cap // 3
    lens = ([edge - 16, edge - 15, edge, cap, 0, 1, cap // 8, cap // 4] * (units // 4 + 1))[:units]
    w = make_custom(1, units, units, cap, d, dtype, seed=35)
    Ka, Va = (dev(x, dtype).reshape(units, cap, d).clone() for x in (w.K, w.V))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(36)
    q = torch.randn((units, d), generator=gen, device=DEV).to(Ka.dtype)
    la = torch.tensor(lens, dtype=torch.int32, device=DEV)
    dm = z.dims_of(None, None, None, B=1, Hq=units, Hkv=units, n=cap, d=d, dtype=1 if dtype == "bf16" else 0)
    size = z.workspace_bytes(z.OP_DECODE, dm)
    assert size == fine * units * (d + 2) * 4
    ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device=DEV)
    o = z.zipvl_decode_attn(q, Ka, Va, la, w.scale, B=1, Hq=units, Hkv=units, ws=ws[:size])
    torch.cuda.synchronize()
    assert int((ws.view(torch.int32) != -1).sum()) == (d + 2) * sum(states(n) for n in lens)
    for u in range(min(units, 8)):
        ref = oz.decode_attention(host64(q[u]), host64(Ka[u]), host64(Va[u]), lens[u], w.scale) if lens[u] else 0.0
        assert np.abs(host64(o[u]) - ref).max() <= ATOL_OUT[dtype]
    # the step that appends the last row of every cache
    lb = torch.clamp(la - 1, min=0)
    kn, vn = (torch.stack([x[u, max(n - 1, 0)] for u, n in enumerate(lens)]) for x in (Ka, Va))
    step_ws = z.decode_step_workspace(1, units, units, cap, d, Ka)
    for _ in range(2):                                        # the arrival counters clear themselves
        ln = lb.clone()
        step = z.zipvl_decode_step(q, Ka, Va, ln, kn, vn, w.scale, B=1, Hq=units, Hkv=units, ws=step_ws)
        torch.cuda.synchronize()
        held = torch.tensor([n > 0 for n in lens], device=DEV)
        assert torch.equal(step[held], o[held]) and ln.tolist() == [max(n, 1) for n in lens]
    assert int(step_ws[:4 * units].view(torch.int32).abs().sum().item()) == 0


@pytest.mark.parametrize("dtype,d,Hq,Hkv", [("bf16", 128, 4, 4), ("bf16", 128, 14, 2), ("f32", 64, 4, 2), ("bf16", 64, 3, 1),
                                            ("f32", 128, 8, 1), ("bf16", 128, 18, 2)])
def test_decode_step_one_launch_matches_append_then_attention(dtype, d, Hq, Hkv):
    """Three consecutive fused steps (the arrival counters must clear themselves) against the oracle's
    append-then-attend, with an empty unit, a long one and one that is full from the second step on."""
    say(f"decode_step dtype={dtype} d={d} Hq={Hq} Hkv={Hkv}")
    B, cap = 2, 1300
    G = Hq // Hkv
    units = B * Hkv
    w = make_custom(B, Hq, Hkv, cap, d, dtype, seed=33)
    Kc = dev(w.K, dtype).reshape(units, cap, d).clone()
    Vc = dev(w.V, dtype).reshape(units, cap, d).clone()
    lens = [0, 1299, 640, 17][:units] + [5] * max(0, units - 4)
    ln = torch.tensor(lens, dtype=torch.int32, device=DEV)
    r = np.random.Generator(np.random.PCG64(34))
    from workloads import round_to_bf16
    cast = round_to_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    Kh = [w.K.reshape(units, cap, d)[u].copy() for u in range(units)]
    Vh = [w.V.reshape(units, cap, d)[u].copy() for u in range(units)]
    ws = z.decode_step_workspace(B, Hq, Hkv, cap, d, Kc)
    worst = 0.0
    for step in range(3):
        q = cast(r.standard_normal((B * Hq, d)).astype(np.float32) * 2)
        kn = cast(r.standard_normal((units, d)).astype(np.float32))
        vn = cast(r.standard_normal((units, d)).astype(np.float32))
        o = z.zipvl_decode_step(dev(q, dtype), Kc, Vc, ln, dev(kn, dtype), dev(vn, dtype), w.scale, B=B, Hq=Hq, Hkv=Hkv, ws=ws)
        torch.cuda.synchronize()
        oh = host64(o)
        new_lens = list(lens)
        for u in range(units):
            if lens[u] < cap:
                Kh[u][lens[u]] = kn[u]; Vh[u][lens[u]] = vn[u]
                new_lens[u] = lens[u] + 1
        for b in range(B):
            for h in range(Hq):
                u = b * Hkv + h // G
                ref = oz.decode_attention(q[b * Hq + h], Kh[u], Vh[u], new_lens[u], w.scale)
                worst = max(worst, np.abs(oh[b * Hq + h] - ref).max())
        lens = new_lens
        assert ln.cpu().tolist() == lens
        for u in range(units):                                # the caches hold exactly the oracle's rows
            assert Kc[u, :lens[u]].to(torch.float32).cpu().numpy().tobytes() == Kh[u][:lens[u]].astype(np.float32).tobytes()
            assert Vc[u, :lens[u]].to(torch.float32).cpu().numpy().tobytes() == Vh[u][:lens[u]].astype(np.float32).tobytes()
    assert int(ws[:4 * units].view(torch.int32).abs().sum().item()) == 0      # counters left at zero
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


@pytest.mark.parametrize("dtype,d,units,G,cap,least,splits", [("bf16", 128, 4, 7, 3900, 16, 16), ("bf16", 128, 2, 7, 4200, 17, 17), ("f32", 128, 3, 2, 8300, 33, 33),
                                                              ("bf16", 64, 1, 8, 17000, 64, 64), ("f32", 64, 1, 5, 300, 2, 2), ("bf16", 64, 64, 2, 24700, 4, 8),
                                                              ("bf16", 64, 32, 3, 49300, 8, 16), ("bf16", 64, 15, 2, 110700, 18, 36),
                                                              ("bf16", 64, 2, 7, 6000, 24, 24), ("bf16", 64, 2, 7, 6200, 25, 25)])
def test_decode_step_of_head_groups_with_few_and_many_splits(dtype, d, units, G, cap, least, splits):
    """The step that merges its splits itself (16 of them at most, 24 for bf16 at d = 64) and the one that leaves it to a second launch, also where a long
    unit has more splits than the others (8 and not 4, 16 and not 8, and in two launches 36 and not 18): empty, short, nearly
    full and full caches, three steps.  The same bits as append and attention one after the other, whose outputs agree with the oracle.
    Which form it was shows in the workspace: of a split with rows a state, of two launches a pair of sums of every split besides."""
    say(f"decode_step of groups dtype={dtype} d={d} units={units} G={G} cap={cap}")
    Hq = units * G
    gen = torch.Generator(device=DEV)
    gen.manual_seed(71)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dt)
    Ka, Va = torch.zeros((units, cap, d), dtype=dt, device=DEV), torch.zeros((units, cap, d), dtype=dt, device=DEV)
    lens = ([cap - 2, 0, 17, cap] + [15, 63, 64, 200] * (units // 4))[:units]
    for u, n in enumerate(lens):
        Ka[u, :n], Va[u, :n] = rnd(n, d), rnd(n, d)
    Kb, Vb, la = Ka.clone(), Va.clone(), torch.tensor(lens, dtype=torch.int32, device=DEV)
    lb = la.clone()
    ws = z.decode_step_workspace(1, Hq, units, cap, d, Ka)
    states = ws[(4 * units + 255) // 256 * 256:].view(torch.int32)

    def splits_of(rows):
        tiles = (rows + 15) // 16
        per = max(1, -(-tiles // (least if tiles <= 384 * least else splits)))
        return max(1, -(-tiles // per))

    scale = 1.0 / math.sqrt(d)
    for step in range(3):
        q, kn, vn = rnd(Hq, d) * 2, rnd(units, d), rnd(units, d)
        states.fill_(-1)
        oa = z.zipvl_decode_step(q, Ka, Va, la, kn, vn, scale, B=1, Hq=Hq, Hkv=units, ws=ws)
        held = sum(splits_of(min(cap, n + 1)) for n in lens)
        assert int((states != -1).sum()) == G * (d * held + 2 * (units * splits if splits > (24 if dtype == "bf16" and d == 64 else 16) else held))
        z.zipvl_kv_append(Kb, Vb, lb, kn, vn, B=1, Hkv=units)
        ob = z.zipvl_decode_attn(q, Kb, Vb, lb, scale, B=1, Hq=Hq, Hkv=units)
        torch.cuda.synchronize()
        assert torch.equal(la, lb) and la.tolist() == [min(cap, n + 1) for n in lens]
        assert torch.equal(oa, ob) and torch.equal(Ka, Kb) and torch.equal(Va, Vb)
        lens = la.tolist()
        for u in range(min(units, 4)):
            for h in (0, G - 1):
                ref = oz.decode_attention(host64(q[u * G + h]), host64(Kb[u]), host64(Vb[u]), lens[u], scale)
                assert np.abs(host64(oa[u * G + h]) - ref).max() <= ATOL_OUT[dtype]
    assert int(ws[:4 * units].view(torch.int32).abs().sum().item()) == 0      # counters left at zero


def test_decode_256_fused_steps_bit_identical_to_append_then_attention_at_the_stack_shape():
    """zipvl_decode_step against zipvl_kv_append + zipvl_decode_attn over 256 consecutive steps at the 32-head,
    batch-4 stack shape: outputs, lengths and caches must agree bit for bit at every step (the fused kernel
    takes the new row in its place in the row order, so the arithmetic is the same).  Lengths are ragged,
    cross split boundaries on the way, one unit starts empty and one fills up and must stay unchanged."""
    say("decode_step x256 vs kv_append + decode_attn, B4 H32 d128")
    B, H, d, cap, steps = 4, 32, 128, 2816, 256
    units = B * H
    g = torch.Generator(device=DEV); g.manual_seed(77)
    Ka = torch.randn((units, cap, d), generator=g, device=DEV).to(torch.bfloat16)
    Va = torch.randn((units, cap, d), generator=g, device=DEV).to(torch.bfloat16)
    r = np.random.Generator(np.random.PCG64(78))
    lens = r.integers(1500, 2500, units).astype(np.int32)
    lens[0], lens[1], lens[2], lens[3] = 0, cap - 100, 255, 2559       # empty; fills up after 100 steps; next to split edges
    la = torch.from_numpy(lens).to(DEV)
    Kb, Vb, lb = Ka.clone(), Va.clone(), la.clone()
    ws = z.decode_step_workspace(B, H, H, cap, d, Ka)
    scale = 1.0 / math.sqrt(d)
    oa = torch.empty((units, d), dtype=torch.bfloat16, device=DEV)
    ob = torch.empty_like(oa)
    for step in range(steps):
        q = torch.randn((units, d), generator=g, device=DEV).to(torch.bfloat16)
        kn = torch.randn((units, d), generator=g, device=DEV).to(torch.bfloat16)
        vn = torch.randn((units, d), generator=g, device=DEV).to(torch.bfloat16)
        z.zipvl_decode_step(q, Ka, Va, la, kn, vn, scale, B=B, Hq=H, Hkv=H, ws=ws, o=oa)
        z.zipvl_kv_append(Kb, Vb, lb, kn, vn, B=B, Hkv=H)
        z.zipvl_decode_attn(q, Kb, Vb, lb, scale, B=B, Hq=H, Hkv=H, o=ob)
        torch.cuda.synchronize()
        if not torch.equal(oa, ob):
            bad = (oa != ob).any(dim=1).nonzero().flatten().tolist()
            raise AssertionError(f"step {step}: outputs differ in units {bad[:8]} (lengths {la[bad[:8]].tolist()})")
        assert torch.equal(la, lb), f"step {step}: lengths differ"
    expect = np.minimum(lens.astype(np.int64) + steps, cap)
    assert la.cpu().numpy().tolist() == expect.tolist()
    assert torch.equal(Ka, Kb) and torch.equal(Va, Vb), "caches differ after 256 steps"
    assert int(ws[:4 * units].view(torch.int32).abs().sum().item()) == 0          # counters left at zero
    # and the last step meets the oracle (Eq. (5)) on a few units, the full one included
    oh = host64(oa)
    for u in (0, 1, 2, 3, 77):
        ref = oz.decode_attention(host64(q[u]), host64(Ka[u]), host64(Va[u]), int(expect[u]), scale)
        assert np.abs(oh[u] - ref).max() <= 2e-2


# B, Hq, Hkv, cap, long length, splits the long units get at least (of at most 3072 rows for one head, 6144 for groups)
UNEQUAL = [(32, 32, 32, 8456, 8192, 3), (16, 32, 32, 8456, 8000, 3), (32, 16, 8, 8456, 8192, 2), (128, 8, 4, 6200, 6145, 2), (1100, 1, 1, 3100, 3073, 2)]


@pytest.mark.parametrize("B,Hq,Hkv,cap,longest,splits", UNEQUAL)
def test_decode_of_unequal_conversations_splits_the_long_one(B, Hq, Hkv, cap, longest, splits):
    """One long conversation (the last of the batch) among short ones and an empty one: its units are shared by several
    workgroups (counted by the partial states that the call leaves in its workspace), the outputs meet the oracle, and
    the fused step gives the same bits, lengths and caches over three steps."""
    say(f"unequal decode B={B} Hq={Hq} Hkv={Hkv} cap={cap}")
    units, d, G = B * Hkv, 64, Hq // Hkv
    g = torch.Generator(device=DEV); g.manual_seed(91)
    Ka = torch.empty((units, cap, d), dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    Va = torch.empty((units, cap, d), dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    lens = np.full(units, 10, dtype=np.int32)
    lens[0], lens[units - Hkv:] = 0, longest
    la, scale = torch.from_numpy(lens).to(DEV), 1.0 / math.sqrt(d)
    q = torch.randn((B * Hq, d), generator=g, device=DEV).to(torch.bfloat16)
    ws = torch.full((z.workspace_bytes(z.OP_DECODE, z.dims_of(None, None, None, B=B, Hq=Hq, Hkv=Hkv, n=cap, d=d, dtype=1)),), 0xFF, dtype=torch.uint8, device=DEV)
    o = z.zipvl_decode_attn(q, Ka, Va, la, scale, B=B, Hq=Hq, Hkv=Hkv, ws=ws)
    torch.cuda.synchronize()
    states = int((ws.view(torch.int32) != -1).sum()) / (G * (d + 2))
    assert states >= (units - Hkv) + Hkv * splits, f"{states} partial states for {units} units"
    oh = host64(o)
    for u in (0, 1, units - Hkv, units - 1):
        ref = oz.decode_attention(host64(q[u * G]), host64(Ka[u]), host64(Va[u]), int(lens[u]), scale) if lens[u] else 0.0
        assert np.abs(oh[u * G] - ref).max() <= 2e-2
    Kb, Vb, lb = Ka.clone(), Va.clone(), la.clone()
    step_ws = z.decode_step_workspace(B, Hq, Hkv, cap, d, Ka)
    for _ in range(3):
        q = torch.randn((B * Hq, d), generator=g, device=DEV).to(torch.bfloat16)
        kn, vn = (torch.randn((units, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
        oa = z.zipvl_decode_step(q, Ka, Va, la, kn, vn, scale, B=B, Hq=Hq, Hkv=Hkv, ws=step_ws)
        z.zipvl_kv_append(Kb, Vb, lb, kn, vn, B=B, Hkv=Hkv)
        ob = z.zipvl_decode_attn(q, Kb, Vb, lb, scale, B=B, Hq=Hq, Hkv=Hkv)
        assert torch.equal(oa, ob) and torch.equal(la, lb)
    assert torch.equal(Ka, Kb) and torch.equal(Va, Vb)
    assert int(step_ws[:4 * units].view(torch.int32).abs().sum().item()) == 0


def test_decode_over_quantised_caches_of_unequal_conversations():
    """Grouped heads: a conversation in a batch where it is by far the longest, against the same conversation alone."""
    say("unequal decode over quantised caches")
    B, Hq, Hkv, n, d, k = 32, 16, 8, 6300, 64, 1500
    g = torch.Generator(device=DEV); g.manual_seed(92)
    K, V = (torch.empty((B, Hkv, n, d), dtype=torch.bfloat16, device=DEV).normal_(generator=g) for _ in range(2))
    idx = torch.arange(n, dtype=torch.int32, device=DEV).repeat(B * Hkv, 1) * 4 % n
    idx[:, :k] = idx[:, :k].sort(dim=1).values
    kc = torch.full((B * Hkv,), k, dtype=torch.int32, device=DEV)
    q = torch.randn((B * Hq, d), generator=g, device=DEV).to(torch.bfloat16)
    all_, one = z.zipvl_quantize_kv(K, V, idx, kc, k, n - k), z.zipvl_quantize_kv(K[:1], V[:1], idx[:Hkv], kc[:Hkv], k, n - k)
    all_.len_hi[Hkv:], all_.len_lo[Hkv:] = 20, 33
    oa = z.zipvl_decode_attn_q(q, all_, 0.125, B=B, Hq=Hq, Hkv=Hkv)
    ob = z.zipvl_decode_attn_q(q[:Hq].contiguous(), one, 0.125, B=1, Hq=Hq, Hkv=Hkv)
    torch.cuda.synchronize()
    # fp32 sums of either split order, rounded to bf16 once: half an ulp of the largest output apart, twice
    assert (oa[:Hq].float() - ob.float()).abs().max() <= 2 ** -8 * ob.float().abs().max()
    assert not torch.isnan(oa.float()).any()


@pytest.mark.parametrize("d,G", [(128, 7), (64, 2)])
@pytest.mark.parametrize("n", [1, 15, 17, 129, 700])
def test_decode_of_head_groups_with_an_infinity_in_v(d, G, n):
    """bf16 groups weigh V with three planes of a weight, of which an infinity makes no number where one is 0: the channel is infinite,
    of its sign, the others agree with the oracle, for a row in the first, the last and a middle tile."""
    say(f"decode of groups with an infinity d={d} G={G} n={n}")
    r = np.random.Generator(np.random.PCG64(n + d))
    K, V, q = (torch.from_numpy(r.standard_normal(s).astype(np.float32)).bfloat16() for s in ((3, n, d), (3, n, d), (3 * G, d)))
    rows = [0, n - 1, n // 2]
    for u in range(3):
        V[u, rows[u], u] = float("inf") if u else -float("inf")
    ln = torch.full((3,), n, dtype=torch.int32, device=DEV)
    o = z.zipvl_decode_attn(q.to(DEV), K.to(DEV), V.to(DEV), ln, d ** -0.5, B=1, Hq=3 * G, Hkv=3)
    torch.cuda.synchronize()
    for u in range(3):
        V[u, rows[u], u] = 0.0
        for h in range(G):
            got = host64(o[u * G + h])
            assert got[u] == (np.inf if u else -np.inf)
            ref = oz.decode_attention(host64(q[u * G + h]), host64(K[u]), host64(V[u]), n, d ** -0.5)
            got[u] = ref[u] = 0.0
            assert np.abs(got - ref).max() <= ATOL_OUT["bf16"]


@pytest.mark.parametrize("dtype,d,G", [("bf16", 128, 7), ("bf16", 64, 2), ("f32", 64, 4), ("f32", 128, 8)])
def test_decode_of_head_groups_at_tile_edges(dtype, d, G):
    """Groups of several heads on the matrix cores (16 cached rows per wave step): lengths on both sides of a tile, of a
    workgroup step and of the capacity, the new row first and last of its tile, NaN in every row that is not part of the
    cache yet.  Fused step against the oracle, and bit for bit against append + attention."""
    say(f"decode tile edges dtype={dtype} d={d} G={G}")
    lens = [0, 1, 14, 15, 16, 17, 127, 128, 255, 256, 511, 599, 600]
    units, cap = len(lens), 600
    w = make_custom(1, units * G, units, cap, d, dtype, seed=35)
    Kc, Vc = dev(w.K, dtype).reshape(units, cap, d).clone(), dev(w.V, dtype).reshape(units, cap, d).clone()
    for u, L in enumerate(lens):
        Kc[u, L:] = float("nan")
        Vc[u, L:] = float("nan")
    g = torch.Generator(device=DEV); g.manual_seed(36)
    dt = Kc.dtype
    q = (2 * torch.randn((units * G, d), generator=g, device=DEV)).to(dt)
    kn, vn = torch.randn((units, d), generator=g, device=DEV).to(dt), torch.randn((units, d), generator=g, device=DEV).to(dt)
    la = torch.tensor(lens, dtype=torch.int32, device=DEV)
    Kb, Vb, lb = Kc.clone(), Vc.clone(), la.clone()
    ws = z.decode_step_workspace(1, units * G, units, cap, d, Kc)
    o = z.zipvl_decode_step(q, Kc, Vc, la, kn, vn, w.scale, B=1, Hq=units * G, Hkv=units, ws=ws)
    z.zipvl_kv_append(Kb, Vb, lb, kn, vn, B=1, Hkv=units)
    ob = z.zipvl_decode_attn(q, Kb, Vb, lb, w.scale, B=1, Hq=units * G, Hkv=units)
    torch.cuda.synchronize()
    assert torch.equal(o, ob) and la.tolist() == lb.tolist() == [min(L + 1, cap) for L in lens]
    assert torch.equal(Kc.view(torch.uint8), Kb.view(torch.uint8)) and torch.equal(Vc.view(torch.uint8), Vb.view(torch.uint8))
    worst = 0.0
    for u, L in enumerate(lens):
        L1 = min(L + 1, cap)
        Kh, Vh = host64(Kc[u, :L1]), host64(Vc[u, :L1])
        for h in range(u * G, u * G + G):
            worst = max(worst, np.abs(host64(o[h]) - oz.decode_attention(host64(q[h]), Kh, Vh, L1, w.scale)).max())
    say(f"  worst |do| = {worst:.3e}")
    assert worst <= ATOL_OUT[dtype]


# ------------------------------------------------------------------ calls without ctypes
def test_calls_of_the_extension_module_are_the_general_ones(monkeypatch):
    """_pycall takes each of the calls; then the same call the general way: the same bits.  Calls that it leaves to the general way, and
    calls that the library refuses: the same errors."""
    say("extension module against ctypes")
    from paper_2410_08584_amd import binding
    binding.load_library()
    module, answers = binding._native, []

    class Recorder:
        def __getattr__(self, name):
            def call(*args):
                answers.append((name, getattr(module, name)(*args)))
                return answers[-1][1]
            return call

    monkeypatch.setattr(binding, "_native", Recorder())
    B, Hq, Hkv, n, d = 2, 4, 2, 500, 64
    w = make_custom(B, Hq, Hkv, n, d, "bf16", seed=81, m=64)
    Q, K, V = (dev(x, "bf16") for x in (w.Q, w.K, w.V))
    units, probes = B * Hkv, [int(p) for p in w.probe_pos]
    new = lambda *shape, dtype=torch.float32: torch.zeros(shape, dtype=dtype, device=DEV)
    byte_ws = lambda nbytes: new(nbytes, dtype=torch.uint8)

    def calls():
        mass, rank, idx, k = new(units, n), new(units, n), new(units, n, dtype=torch.int32), new(units, dtype=torch.int32)
        z.zipvl_score(Q, K, probes, w.scale, mass=mass, rank=rank, ws=byte_ws(z.workspace_bytes(z.OP_SCORE, z.dims_of(Q, K), 64)))
        z.zipvl_select(mass, rank, 0.975, idx=idx, k=k)
        cap = n + 8
        Kc, Vc, ln = new(units, cap, d, dtype=Q.dtype), new(units, cap, d, dtype=Q.dtype), new(units, dtype=torch.int32)
        z.zipvl_compact_kv(K, V, idx, k, cap, Kc=Kc, Vc=Vc, length=ln)
        O = new(B, Hq, n, d, dtype=Q.dtype)
        z.zipvl_sparse_prefill(Q, K, V, idx, k, w.scale, O=O, ws=byte_ws(z.workspace_bytes(z.OP_SPARSE_PREFILL, z.dims_of(Q, K, V))))
        q, kn, vn = Q[:, :, 3].reshape(B * Hq, d).contiguous(), K[:, :, 3].reshape(units, d).contiguous(), V[:, :, 3].reshape(units, d).contiguous()
        o = new(B * Hq, d, dtype=Q.dtype)
        z.zipvl_decode_step(q, Kc, Vc, ln, kn, vn, w.scale, B=B, Hq=Hq, Hkv=Hkv, ws=z.decode_step_workspace(B, Hq, Hkv, cap, d, Kc), o=o)
        cache = z.zipvl_quantize_kv(K, V, idx, k, n, n)
        Kt, Vt, lt, oq = new(units, 9, d, dtype=Q.dtype), new(units, 9, d, dtype=Q.dtype), new(units, dtype=torch.int32), new(B * Hq, d, dtype=Q.dtype)
        z.zipvl_kv_append(Kt, Vt, lt, kn, vn, B=B, Hkv=Hkv)
        dq = z.dims_of(None, None, None, B=B, Hq=Hq, Hkv=Hkv, n=2 * n + 9, d=d, dtype=1)
        z.zipvl_decode_attn_q(q, cache, w.scale, B=B, Hq=Hq, Hkv=Hkv, K_tail=Kt, V_tail=Vt, len_tail=lt, o=oq, ws=byte_ws(z.workspace_bytes(z.OP_DECODE_Q, dq)))
        torch.cuda.synchronize()
        kept = [idx[u, : int(k[u])] for u in range(units)]
        return [mass, rank, k, ln, O, o, Kt, Vt, lt, oq, *kept, *(Kc[u, : int(ln[u])] for u in range(units))]

    def refusals():
        ws, mass = byte_ws(1 << 20), new(units, n)
        cap = 16
        Kc, ln, o, x = new(units, cap, d, dtype=Q.dtype), new(units, dtype=torch.int32), new(B * Hq, d, dtype=Q.dtype), new(units, d, dtype=Q.dtype)
        bad = [lambda: z.zipvl_score(Q, K, probes[::-1], w.scale, mass=mass, rank=mass, ws=ws),
               lambda: z.zipvl_score(Q, K, probes, w.scale, mass=mass, rank=mass, ws=ws[:256]),
               lambda: z.zipvl_score(Q, K, probes, -1.0, mass=mass, rank=mass, ws=ws),
               lambda: z.zipvl_score(Q.half(), K, probes, w.scale, mass=mass, rank=mass, ws=ws),
               lambda: z.zipvl_score(Q.transpose(2, 3), K, probes, w.scale, mass=mass, rank=mass, ws=ws),
               lambda: z.zipvl_score(Q, K, probes, w.scale, mass=mass.t(), rank=mass, ws=ws),
               lambda: z.zipvl_select(mass, mass, 2.0, idx=new(units, n, dtype=torch.int32), k=ln, ws=ws[:8]),
               lambda: z.zipvl_sparse_prefill(Q, K, V, None, ln, w.scale, O=torch.empty_like(Q), ws=ws),
               lambda: z.zipvl_compact_kv(K, V, None, ln, 0, Kc=Kc, Vc=Kc, length=ln),
               lambda: z.zipvl_kv_append(Kc, Kc, ln, x, x, B=-1, Hkv=Hkv),
               lambda: z.zipvl_decode_step(o, Kc, Kc, ln, x, x, w.scale, B=B, Hq=3, Hkv=2, ws=ws, o=o),
               lambda: z.zipvl_decode_step(o, Kc[0], Kc, ln, x, x, w.scale, B=B, Hq=Hq, Hkv=Hkv, ws=ws, o=o)]
        out = []
        for call in bad:
            with pytest.raises(Exception) as e:
                call()
            out.append((type(e.value), str(e.value)))
        return out

    direct = calls()
    assert sorted(answers) == [(name, 0) for name in ("compact_kv", "decode_attn_q", "decode_step", "kv_append", "score", "select", "sparse_prefill")]
    answers.clear()
    refused = refusals()
    # the library's own refusals; None: dtype, strides or shape that the general way handles
    taken = [("score", True)] * 3 + [("score", False)] * 3 + [("select", True), ("sparse_prefill", True), ("compact_kv", True), ("kv_append", True),
                                                                ("decode_step", True), ("decode_step", False)]
    assert [(name, rc is not None) for name, rc in answers] == taken and all(rc is None or rc < 0 for _, rc in answers)
    took = []

    class General:
        def __getattr__(self, name):
            return lambda *a: took.append(name)

    monkeypatch.setattr(binding, "_native", General())
    for a, b in zip(direct, calls()):
        assert torch.equal(a, b)
    assert sorted(set(took)) == ["compact_kv", "decode_attn_q", "decode_step", "kv_append", "score", "select", "sparse_prefill"]
    assert refused == refusals()

"""Fair draws from weighted samples on the GPU: indices bit-exact against the
oracle (integer masses and prefix sums on both sides) on a ragged sample
count with non-finite weights, the drawn samples copied out, the no-weight
case, and the resampling check on an ILE run: the fair draws reproduce the
weighted distribution of the run's samples in every column."""
import numpy as np
import pytest

import chirpgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2505_11655_amd as ile  # noqa: E402
from tests import gpu_util as gu  # noqa: E402


def _job(policy, seed=110):
    rng = np.random.default_rng(seed)
    p = chirpgen.random_problem(rng, 5, ["H", "L"])
    return ile.ile_prepare(gu.ctx(), ile.ProblemHost(p, precision=policy))


@pytest.mark.parametrize("policy", [ile.ILE_FP64, ile.ILE_FP32, ile.ILE_FP32_CANCEL64],
                         ids=["fp64", "fp32", "fp32c64"])
@pytest.mark.parametrize("n", [1, 4095, 100003])
def test_fair_draw_matches_oracle(orc, policy, n):
    rng = np.random.default_rng(111 + n)
    lw = rng.normal(0, 4, n)
    if n > 10:
        lw[rng.choice(n, n // 20, replace=False)] = -np.inf
        lw[rng.choice(n, 3, replace=False)] = np.nan
        lw[5] = lw[np.isfinite(lw)].max()          # a tie at the maximum
    odt = np.float32 if policy == ile.ILE_FP32 else np.float64
    tdt = np.float64 if policy == ile.ILE_FP64 else np.float32
    lw = lw.astype(odt)
    th = rng.normal(size=(7, n)).astype(tdt)
    k = 30011
    job = _job(policy)
    try:
        lw_d = torch.from_numpy(lw).to("cuda")
        th_d = torch.from_numpy(th).to("cuda")
        idx = torch.full((k,), -7, dtype=torch.int64, device="cuda")
        out = torch.zeros((7, k), dtype=th_d.dtype, device="cuda")
        ile.ile_fair_draw(job, n, lw_d, 0xFA1, 4, k, idx, th_d, n, out, k)
        torch.cuda.synchronize()
        g = idx.cpu().numpy()
    finally:
        ile.ile_job_release(job)
    o = orc.fair_draw(lw.astype(np.float64), 0xFA1, 4, k)
    assert np.array_equal(g, o)
    assert np.array_equal(out.cpu().numpy(), th[:, o])


@pytest.mark.parametrize("n,spread,shift", [
    (63, 1.0, 0), (64, 1.0, 1), (65, 0.0, 0),           # one granule of 64 samples and its edges
    (4096, 2.0, 1), (4097, 2.0, 3),                     # one tile, and a second one of one sample
    (2048 * 4096 + 1, 9.0, 1),                          # more tiles than runs: two tiles per run
])
def test_fair_draw_granules_tiles_runs(orc, n, spread, shift):
    """Indices equal to the oracle's at the edges of the granules, tiles and
    runs that the masses are summed by, from a buffer that starts `shift`
    values past an aligned address, with infinities of both signs."""
    rng = np.random.default_rng(113 + n)
    lw = rng.normal(0, spread, n).astype(np.float32)
    lw[rng.choice(n, 2, replace=False)] = [np.inf, -np.inf]
    job = _job(ile.ILE_FP32, seed=114)
    k = 5003
    try:
        buf = torch.zeros(n + shift, dtype=torch.float32, device="cuda")
        buf[shift:] = torch.from_numpy(lw).to("cuda")
        idx = torch.full((k,), -7, dtype=torch.int64, device="cuda")
        ile.ile_fair_draw(job, n, buf.data_ptr() + 4 * shift, 0xFA2, 5, k, idx)
        torch.cuda.synchronize()
    finally:
        ile.ile_job_release(job)
    lw = np.where(np.isfinite(lw), lw, -np.inf).astype(np.float64)
    assert np.array_equal(idx.cpu().numpy(), orc.fair_draw(lw, 0xFA2, 5, k))


@pytest.mark.parametrize("n,k", [(20011, 20011), ((1 << 23) + 5, 70001)])
@pytest.mark.parametrize("out", ["idx", "theta"])
def test_fair_draw_over_its_weights(orc, out, n, k):
    """Outputs that lie over the log-weights: the indices in their place, or a
    column of the drawn samples, with a prefix per sample and with one per 64
    samples (whose picks read the weights again).  As from separate buffers."""
    rng = np.random.default_rng(116)
    lw = rng.normal(0, 2.0, n)
    job = _job(ile.ILE_FP64, seed=117)
    ref = orc.fair_draw(lw, 0xFA3, 6, k)
    try:
        buf = torch.zeros(3 * n, dtype=torch.float64, device="cuda")
        w = buf[n:2 * n]
        w[:] = torch.from_numpy(lw).to("cuda")
        if out == "idx":
            idx = w[n - k:].view(torch.int64)
            ile.ile_fair_draw(job, n, w, 0xFA3, 6, k, idx)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), ref)
        else:
            th = rng.normal(size=(7, n))
            theta = torch.from_numpy(th).to("cuda")
            o = buf[n - k:]   # its second column begins where the weights do
            if o.numel() < 7 * k:
                buf = torch.cat([buf, torch.zeros(7 * k, dtype=torch.float64, device="cuda")])
                w, o = buf[n:2 * n], buf[n - k:]
            ile.ile_fair_draw(job, n, w, 0xFA3, 6, k, None, theta, n, o, k)
            torch.cuda.synchronize()
            assert np.array_equal(o[:7 * k].view(7, k).cpu().numpy(), th[:, ref])
    finally:
        ile.ile_job_release(job)


@pytest.mark.parametrize("n,k", [((3 << 19), 3001), ((3 << 19) + 1, 3001), ((1 << 23) + 4097, (1 << 19) + 257)])
def test_fair_draw_prefix_rule(orc, n, k):
    """Both sides of the rule for the prefixes (per sample up to 1.5 x 2^20 samples and
    for more than a draw per 16 samples, else per 64 samples): the oracle's
    indices, and the same where the context's budget holds only the smaller
    scratch."""
    rng = np.random.default_rng(118)
    lw = rng.normal(0, 3.0, n).astype(np.float32)
    lw[: n // 3] = -np.inf
    ref = orc.fair_draw(lw.astype(np.float64), 0xFA4, 7, k)
    lw_d = torch.from_numpy(lw).to("cuda")
    for budget in (0, 48 << 20 if n > 1 << 23 else 8 << 20):
        ctx = ile.ile_ctx_create(0, budget)
        job = ile.ile_prepare(ctx, ile.ProblemHost(chirpgen.random_problem(rng, 5, ["H", "L"]), precision=ile.ILE_FP32))
        try:
            idx = torch.full((k,), -7, dtype=torch.int64, device="cuda")
            ile.ile_fair_draw(job, n, lw_d, 0xFA4, 7, k, idx)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), ref)
        finally:
            ile.ile_job_release(job)
            ile.ile_ctx_destroy(ctx)


def test_fair_draw_capture_after_fewer_draws(orc):
    """A graph captured after a call with few draws (prefixes by 64 samples) may
    ask for many: it takes the scratch that is there.  Replays with other
    work in between equal the oracle."""
    rng = np.random.default_rng(119)
    n, k = (1 << 23) + 4097, (1 << 19) + 257
    lw = rng.normal(0, 3.0, n).astype(np.float32)
    ref = orc.fair_draw(lw.astype(np.float64), 0xFA5, 8, k)
    lw_d = torch.from_numpy(lw).to("cuda")
    job = _job(ile.ILE_FP32, seed=120)
    try:
        st = torch.cuda.Stream()
        idx = torch.full((k,), -7, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            ile.ile_fair_draw(job, n, lw_d, 0xFA5, 8, 1000, idx, stream=st.cuda_stream)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            ile.ile_fair_draw(job, n, lw_d, 0xFA5, 8, k, idx, stream=st.cuda_stream)
        for _ in range(3):
            idx.fill_(-7)
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), ref)
            (lw_d * 2).sum().item()
        del g
    finally:
        ile.ile_job_release(job)


def test_fair_draw_without_weight_and_errors():
    job = _job(ile.ILE_FP64, seed=112)
    try:
        lw = torch.full((100,), float("-inf"), dtype=torch.float64, device="cuda")
        th = torch.zeros((7, 100), dtype=torch.float64, device="cuda")
        idx = torch.zeros(50, dtype=torch.int64, device="cuda")
        out = torch.zeros((7, 50), dtype=torch.float64, device="cuda")
        ile.ile_fair_draw(job, 100, lw, 1, 0, 50, idx, th, 100, out, 50)
        torch.cuda.synchronize()
        assert np.all(idx.cpu().numpy() == -1) and torch.isnan(out).all().item()
        with pytest.raises(ile.IleError):
            ile.ile_fair_draw(job, 0, lw, 1, 0, 5, idx)
        with pytest.raises(ile.IleError):
            ile.ile_fair_draw(job, 100, lw, 1, 0, 5, None, th, 100, out, 4)
    finally:
        ile.ile_job_release(job)


def test_fair_draws_reproduce_the_weighted_run():
    """Before/after resampling: prior draws of an SNR-10 HL event weighted by
    the FP64 likelihood, then 20,000 fair draws; the draw counts of the
    samples follow their weights (chi-square over the samples with expected
    count >= 5, the rest pooled), and each column's mean over the draws
    agrees with the weighted mean within 5 standard errors."""
    from scipy import stats
    rec = chirpgen.load_injections()["pool"][7]
    probs, _ = chirpgen.build_event(rec, ["H", "L"], 5, 25.0, 1.5, 10.0, noise_seed=77)
    job = ile.ile_prepare(gu.ctx(), ile.ProblemHost(probs[0], precision=ile.ILE_FP64))
    n, k = 1 << 21, 20000
    try:
        th = torch.empty((7, n), dtype=torch.float64, device="cuda")
        lr = torch.empty((n,), dtype=torch.float64, device="cuda")
        L = torch.empty((n,), dtype=torch.float64, device="cuda")
        W = torch.empty((n,), dtype=torch.float64, device="cuda")
        ile.ile_draw(job, 31, 0, 0, n, th, n, lr)
        ile.ile_eval_lnL(job, n, th, n, lr, L, W)
        m = ile.ile_marginalize(job, n, W)
        idx = torch.empty(k, dtype=torch.int64, device="cuda")
        out = torch.empty((7, k), dtype=torch.float64, device="cuda")
        ile.ile_fair_draw(job, n, W, 32, 0, k, idx, th, n, out, k)
        torch.cuda.synchronize()
        w = W.cpu().numpy()
        x = th.cpu().numpy()
        d = out.cpu().numpy()
        ix = idx.cpu().numpy()
    finally:
        ile.ile_job_release(job)
    print("n_eff", m["n_eff"])
    w = np.exp(w - w.max())
    p = w / w.sum()
    big = np.nonzero(p * k >= 5)[0]
    cnt = np.array([np.count_nonzero(ix == i) for i in big] + [np.count_nonzero(~np.isin(ix, big))])
    exp_ = np.concatenate([p[big] * k, [k * (1 - p[big].sum())]])
    keep = exp_ > 0
    assert stats.chisquare(cnt[keep], exp_[keep] / exp_[keep].sum() * cnt[keep].sum()).pvalue > 1e-4
    assert np.array_equal(d, x[:, ix])
    for c in range(7):
        mu = float(np.sum(p * x[c]))
        sd = float(np.sqrt(np.sum(p * (x[c] - mu) ** 2)))
        assert abs(d[c].mean() - mu) <= 5 * sd / np.sqrt(k) + 1e-12, c

"""GPU parity of the softmax statistics, Algorithm 1 and the accept/resample
walk against the oracle, on shared seeded logits (called through the C ABI).

Decisions (accepted rows, branch, emitted token, flags) must be bit-exact
given the same uniforms, except where the oracle's own path passes within
1e-6 of a threshold (|u - p~/q| or |u*W - C_v| / W), where summation order
and exp ulps may legitimately flip a decision.
"""
import ctypes as C
import json
import os

import numpy as np
import pytest
import torch

from gpu_util import decision_margin, say
from oracle import sampling, tree
from paper_2506_01979_amd import synth

pytestmark = pytest.mark.gpu

TIE = 1e-6


@pytest.fixture(scope="module")
def api():
    from paper_2506_01979_amd import api as A
    assert torch.cuda.is_available()
    return A


def dev(x, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(x))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


@pytest.mark.parametrize("vocab", [16, 1000, 32000, 128256])
@pytest.mark.parametrize("T", [1.0, 0.7, 0.0])
def test_softmax_stats(api, vocab, T):
    say(f"stats vocab={vocab} T={T}")
    n = 5
    lg = synth.random_logits(n, vocab, 3.0, seed=vocab)
    lg[1, 7] = lg[1].max() + 1.0          # a clear max
    lg[2, [3, 9]] = lg[2].max() + 0.5     # a tie: lowest index wins
    st = api.new_stats(n)
    api.sb_softmax_stats(dev(lg), T, st)
    torch.cuda.synchronize()
    got = api.decode_stats(st)
    for i in range(n):
        ref = sampling.row_stats(lg[i], T)
        assert got["argmax"][i] == ref.argmax
        assert np.float32(got["zmax"][i]) == np.float32(ref.zmax)
        assert abs(got["total"][i] - ref.total) <= 1e-6 * ref.total


def test_softmax_stats_nonfinite(api):
    lg = synth.random_logits(3, 100, 1.0)
    lg[0, 5] = np.nan
    lg[1, 6] = np.inf
    lg[2, 7] = -np.inf      # a masked token is not an error
    st = api.new_stats(3)
    api.sb_softmax_stats(dev(lg), 1.0, st)
    got = api.decode_stats(st)
    assert np.isnan(got["total"][0]) and np.isnan(got["total"][1])
    assert np.isfinite(got["total"][2])


def _golden():
    p = os.path.join(os.path.dirname(__file__), "golden", "accept_cases.txt")
    with open(p) as f:
        return [json.loads(l) for l in f if l.strip() and not l.startswith("#")]


@pytest.mark.parametrize("case", _golden(), ids=lambda c: c["name"])
def test_select_golden(api, case):
    say(f"select golden {case['name']}")
    p = np.asarray(case["p"], dtype=np.float64)
    lg = np.where(p > 0, np.log(np.maximum(p, 1e-300)), -1e30).astype(np.float32)
    V = len(p)
    st = api.new_stats(1)
    api.sb_softmax_stats(dev(lg[None]), 1.0, st)
    q = np.asarray(case["q"], dtype=np.float32)
    out = torch.zeros(3, dtype=torch.int32, device="cuda")
    ws = torch.empty(api.sb_sample_workspace_bytes(V), dtype=torch.uint8, device="cuda")
    api.sb_select_branch(dev(lg), st, 1.0, dev(np.asarray(case["x"], np.int32)), dev(q),
                         dev(np.asarray(case["u"], np.float32)), out, ws)
    o = out.cpu().numpy()
    assert int(o[0]) == case["accepted"]
    assert int(o[1]) == case["token"]


@pytest.mark.parametrize("vocab,n_cand,T", [(1000, 1, 1.0), (1000, 3, 1.0), (32000, 4, 1.0),
                                            (32000, 6, 0.8), (32000, 3, 0.0), (128256, 4, 1.0)])
def test_select_random(api, vocab, n_cand, T):
    say(f"select random vocab={vocab} n_cand={n_cand} T={T}")
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    out = torch.zeros(3, dtype=torch.int32, device="cuda")
    checked = 0
    for seed in range(12):
        lg = synth.random_logits(1, vocab, 2.0, seed=100 + seed)[0]
        pst = sampling.row_stats(lg, T)
        p = sampling.target_probs(lg, T, pst)
        qr = synth.softmax_rows(synth.random_logits(1, vocab, 2.0, seed=200 + seed))[0]
        # q partly aligned with p so that acceptances and rejections both occur
        qa = (0.5 * p + 0.5 * qr).astype(np.float32)
        q = np.stack([qa] * n_cand)
        g = np.random.default_rng(seed)
        toks = np.array([g.choice(vocab, p=qa / qa.sum()) for _ in range(n_cand)], np.int32)
        u = synth.uniforms(n_cand + 1, seed=300 + seed)
        tr = []
        res = sampling.branch_select(p, toks, q, u[:n_cand], trace=tr)
        if res.accepted is None:
            y = sampling.draw(res.p_tilde, float(u[n_cand]), tr, n_cand)
            want = (-1, y, res.flags)
        else:
            want = (res.accepted, int(toks[res.accepted]), res.flags)
        st = api.new_stats(1)
        api.sb_softmax_stats(dev(lg[None]), T, st)
        api.sb_select_branch(dev(lg), st, T, dev(toks), dev(q), dev(u), out, ws)
        got = tuple(int(x) for x in out.cpu().numpy())
        if decision_margin(tr, u) < TIE:
            continue
        assert got == want, (seed, got, want)
        checked += 1
    assert checked >= 10


def _walk_case(vocab, parents, T, alpha, seed):
    """Seeded logits, q rows (alpha * p(parent) + (1 - alpha) * q_rand) and
    draft tokens drawn from q."""
    n = len(parents)
    lg = synth.random_logits(n, vocab, 2.0, seed=seed)
    p = np.stack([sampling.target_probs(lg[i], T) for i in range(n)])
    qr = synth.softmax_rows(synth.random_logits(n, vocab, 2.0, seed=seed + 1))
    q = np.zeros((n, vocab), dtype=np.float32)
    g = np.random.default_rng(seed)
    toks = np.zeros(n, dtype=np.int32)
    toks[0] = g.integers(0, vocab)
    for i in range(1, n):
        row = (alpha * p[parents[i]] + (1 - alpha) * qr[i]).astype(np.float32)
        q[i] = row
        toks[i] = g.choice(vocab, p=row.astype(np.float64) / row.astype(np.float64).sum())
    u = synth.uniforms(n, seed=seed + 2)
    return lg, q, toks, u


def _random_tree(n, seed):
    g = np.random.default_rng(seed)
    par = [-1] + [int(g.integers(0, i)) for i in range(1, n)]
    return np.asarray(par, dtype=np.int32)


TREES = [
    ("b4k8", synth.branch_parents(4, 8)),
    ("b1k4", synth.branch_parents(1, 4)),
    ("b8k16", synth.branch_parents(8, 16)),
    ("b2k1", synth.branch_parents(2, 1)),
    ("chain20", synth.chain_parents(20)),
    ("fork4x4x7", synth.fork_parents(4, 4, 7)),
    ("fork6x5x1", synth.fork_parents(6, 5, 1)),
    ("random60", _random_tree(60, 3)),
    ("root_only", np.array([-1], dtype=np.int32)),
    # SB_MAX_ROWS = 256 rows: 15 branches of 17, and a random tree
    ("b15k17", synth.branch_parents(15, 17)),
    ("random256", _random_tree(256, 7)),
]


@pytest.mark.parametrize("name,parents", TREES, ids=[t[0] for t in TREES])
@pytest.mark.parametrize("vocab,T", [(1000, 1.0), (32000, 1.0), (32000, 0.0), (4096, 0.6)])
def test_walk_parity(api, name, parents, vocab, T):
    n = len(parents)
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    res_t = api.new_result()
    checked = 0
    outcomes = set()
    cases = 8
    for k in range(cases):
        alpha = (0.2, 0.6, 0.9, 0.99)[k % 4]
        seed = 1000 * k + n + vocab
        say(f"walk {name} vocab={vocab} T={T} case={k} seed={seed}")
        lg, q, toks, u = _walk_case(vocab, parents, T, alpha, seed)
        tr = []
        ref = sampling.accept_resample(toks, parents, lg, T, q, u, trace=tr)
        st = api.new_stats(n)
        dl = dev(lg)
        api.sb_softmax_stats(dl, T, st)
        api.sb_accept_resample(dev(toks), parents, dl, st, T, dev(q), dev(u), res_t, ws)
        got = api.decode_result(res_t)
        if decision_margin(tr, u) < TIE:
            continue
        assert got["path"] == ref.path, (k, got, ref)
        assert got["n_accepted"] == ref.n_accepted
        assert got["branch"] == ref.branch
        assert got["next_token"] == ref.next_token
        assert got["flags"] == ref.flags
        assert got["n_rejected"] == ref.n_rejected
        assert bool(got["bonus"]) == ref.bonus
        outcomes.add((ref.n_accepted, ref.bonus))
        checked += 1
    assert checked >= cases - 2


@pytest.mark.parametrize("vocab,T", [(1023, 1.0), (1024, 1.0), (1025, 0.8), (2047, 0.0), (65536, 1.0),
                                     (65537, 0.7), (131073, 1.0), (270001, 1.0), (2097153, 1.0)])
def test_select_slices(api, vocab, T):
    """Selections that reject up to three candidates and accept one, at the
    edges of the vocabulary slices a workgroup holds (one workgroup, a slice of
    one token, each slice width, a width not a multiple of 4, and the form in
    memory past the slices' reach); one row is twice the distribution it
    tests, which leaves a residual without mass.  test_select_draws has those
    that reject all."""
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    out = torch.zeros(3, dtype=torch.int32, device="cuda")
    for seed in range(6 if vocab < 1000000 else 2):
        say(f"select slices vocab={vocab} T={T} seed={seed}")
        lg = synth.random_logits(1, vocab, 2.0, seed=500 + seed)[0]
        p = sampling.target_probs(lg, T, sampling.row_stats(lg, T))
        qr = synth.softmax_rows(synth.random_logits(1, vocab, 2.0, seed=600 + seed))[0]
        qa = (0.4 * p + 0.6 * qr).astype(np.float32)
        q = np.stack([qa, qr, qa, qr])
        if seed % 2:
            q[seed // 2 % 2] = (2.0 * p).astype(np.float32)
        g = np.random.default_rng(seed)
        toks = g.integers(0, vocab, 4).astype(np.int32)
        toks[3] = np.argmax(p)
        u = np.array([0.9, 0.97, 0.9, 0.5, synth.uniforms(1, seed=700 + seed)[0]], np.float32)
        tr = []
        res = sampling.branch_select(p, toks, q, u[:4], trace=tr)
        assert res.accepted is not None
        want = (res.accepted, int(toks[res.accepted]), res.flags)
        st = api.new_stats(1)
        api.sb_softmax_stats(dev(lg[None]), T, st)
        api.sb_select_branch(dev(lg), st, T, dev(toks), dev(q), dev(u), out, ws)
        got = tuple(int(x) for x in out.cpu().numpy())
        assert decision_margin(tr, u) > TIE
        assert got == want, (seed, got, want)


def _slice_tokens(vocab):
    """Tokens of one workgroup's slice of the vocabulary (k_walk.hip)."""
    per = 1024
    while per < 8192 and -(-vocab // per) > 64:
        per *= 2
    return per


def _all_rejected(vocab, n, T, seed):
    """A target row and n candidates that are far likelier under their own
    rows than under it, tested with u = 0.9: every one is rejected.  The last
    token is a likely one (it may be a slice of its own)."""
    lg = synth.random_logits(1, vocab, 2.0, seed=seed)[0]
    lg[-1] = lg.max()
    p = sampling.target_probs(lg, T)
    q = synth.softmax_rows(synth.random_logits(n, vocab, 2.0, seed=seed + 1)).astype(np.float32)
    toks = np.argmax(q - 20.0 * p, axis=1).astype(np.int32)
    return lg, p, q, toks, np.full(n, 0.9, np.float32)


def _uniform_into(pt, lo, hi):
    """The uniform whose draw from the weights pt is the heaviest of tokens
    lo .. hi - 1, in the middle of its range."""
    c = np.cumsum(pt)
    y = lo + int(np.argmax(pt[lo:hi]))
    return np.float32((c[y] - 0.5 * pt[y]) / c[-1])


@pytest.mark.parametrize("vocab", [2049, 5000, 70001])
@pytest.mark.parametrize("walk", [False, True])
def test_walk_gives_up(api, vocab, walk):
    """Workgroups that do not wait for a message (forced from the host; every
    kernel ends normally) leave a whole and right result, whichever they are:
    workgroup 0, the one whose slice the draw crosses, every other, all; from
    each exchange on.  The result holds a sentinel before every call."""
    name = "sb_internal_" + ("accept_resample" if walk else "select_branch")
    f = getattr(api.lib, name)
    f.restype = C.c_int32
    f.argtypes = (api.lib.sb_accept_resample if walk else api.lib.sb_select_branch).argtypes + [C.c_uint64] + [C.c_int32] * 3
    per = _slice_tokens(vocab)
    G = -(-vocab // per)
    n = 3
    lg, p, q, toks, u = _all_rejected(vocab, n, 1.0, vocab)
    pt = sampling.branch_select(p, toks, q, u).p_tilde
    st = api.new_stats(n + 1)
    rows = np.stack([lg] * (n + 1))
    dl = dev(rows)
    api.sb_softmax_stats(dl, 1.0, st)
    ws = torch.full((api.sb_sample_workspace_bytes(vocab),), 0x5a, dtype=torch.uint8, device="cuda")
    dt = dev(np.concatenate([[0], toks]).astype(np.int32))
    dq = dev(np.concatenate([q[:1], q]))
    par = np.array([-1] + [0] * n, np.int32)
    for owner in sorted({0, G // 2, G - 1}):
        uf = _uniform_into(pt, owner * per, min(vocab, (owner + 1) * per))
        tr = []
        ref = sampling.accept_resample(np.concatenate([[0], toks]), par, rows, 1.0, np.concatenate([q[:1], q]),
                                       np.concatenate([[uf], u]), trace=tr)
        assert ref.n_rejected == n and ref.next_token // per == owner
        assert decision_margin(tr, np.concatenate([[uf], u])) > TIE
        du = dev(np.concatenate([[uf], u]) if walk else np.concatenate([u, [uf]]))
        for lo, hi in [(0, 0), (0, 1), (owner, owner + 1), (1, G), (0, G)]:
            for at in range(n + 1):
                say(f"{name} vocab={vocab} owner={owner} gives up {lo}..{hi} from {at}")
                out = torch.full((264,), -7, dtype=torch.int32, device="cuda")
                tail = (du.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), api._stream(), 100000, lo, hi, at)
                if walk:
                    rc = f(vocab, n + 1, dt.data_ptr(), par.ctypes.data_as(C.POINTER(C.c_int32)), dl.data_ptr(),
                           st.data_ptr(), 1.0, dq.data_ptr(), *tail)
                else:
                    rc = f(vocab, dl.data_ptr(), st.data_ptr(), 1.0, n, dt[1:].data_ptr(), dq[1:].data_ptr(), *tail)
                assert rc == 0
                o = out.cpu().numpy()
                if walk:
                    got = api.decode_result(out)
                    assert got["next_token"] == ref.next_token, (lo, hi, at)
                    assert got["path"] == [0] and got["n_accepted"] == 0 and got["branch"] == -1
                    assert (got["flags"], got["n_rejected"], got["bonus"]) == (0, n, 0)
                else:
                    assert o[:3].tolist() == [-1, ref.next_token, 0], (lo, hi, at)


@pytest.mark.parametrize("vocab", [64, 5000, 70001])
@pytest.mark.parametrize("bad", ["nan first", "nan last", "inf", "marked"])
@pytest.mark.parametrize("T", [1.0, 0.0])
def test_walk_nonfinite_row(api, vocab, bad, T):
    """A row that is not finite has no mass at T > 0: the draw from it is the
    last token, wherever the NaN or infinity stands, and also where only its
    total says so (a forward that was not valid); at T = 0 it is its argmax.
    By the workgroups together and by workgroup 0 alone, with no candidate
    (the bonus draw) and after two rejections."""
    lg, p, q, toks, u = _all_rejected(vocab, 2, 1.0, 40 + vocab)
    lg[-1] = lg.min()  # not the argmax
    if bad.startswith("nan"):
        lg[3 if bad == "nan first" else vocab - 2] = np.nan
    elif bad == "inf":
        lg[vocab // 2] = np.inf
    ref_st = sampling.row_stats(lg, T)
    st = api.new_stats(3)
    rows = np.stack([lg] * 3)
    dl = dev(rows)
    api.sb_softmax_stats(dl, T, st)
    if bad == "marked":
        ref_st.total = float("nan")
        st.view(torch.float64)[:, 1] = float("nan")
    stats = [ref_st] * 3
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    f = api.lib.sb_internal_accept_resample
    f.restype = C.c_int32
    f.argtypes = api.lib.sb_accept_resample.argtypes + [C.c_uint64] + [C.c_int32] * 3
    tok3, q3 = np.concatenate([[0], toks]).astype(np.int32), np.concatenate([q[:1], q])
    u3 = np.concatenate([[0.4], u]).astype(np.float32)
    dt, dq, du = dev(tok3), dev(q3), dev(u3)
    for n in (1, 3):
        par = np.array([-1, 0, 0][:n], np.int32)
        with np.errstate(invalid="ignore"):
            ref = sampling.accept_resample(tok3, par, rows, T, q3, u3, stats=stats)
        if T > 0:
            assert ref.next_token == vocab - 1
        for hi in (0, 1):
            say(f"non-finite row vocab={vocab} {bad} T={T} n={n} gives up 0..{hi}")
            out = api.new_result()
            assert f(vocab, n, dt.data_ptr(), par.ctypes.data_as(C.POINTER(C.c_int32)), dl.data_ptr(), st.data_ptr(), T,
                     dq.data_ptr(), du.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), api._stream(), 100000, 0, hi,
                     0) == 0
            got = api.decode_result(out)
            assert got["next_token"] == ref.next_token
            assert got["flags"] == ref.flags and got["flags"] & api.SB_FLAG_NONFINITE
            assert (got["n_rejected"], bool(got["bonus"])) == (ref.n_rejected, ref.bonus)


def _four_rejected(vocab, seed):
    """As _all_rejected with four candidates, the second one's row twice the
    distribution it is tested against, which leaves a residual without mass;
    the third one's ratio is 0.8."""
    lg, p, q, toks, u = _all_rejected(vocab, 4, 1.0, seed)
    pt = sampling.branch_select(p, toks[:1], q[:1], u[:1]).p_tilde
    q[1] = (2.0 * pt).astype(np.float32)
    toks[1] = toks[2] = np.argmax(pt[:-1])
    q[2, toks[2]] = pt[toks[2]] / 0.8
    return lg, p, q, toks, u


@pytest.mark.parametrize("vocab", [1000, 1025, 2048, 2049, 4096, 4097, 65536, 65537, 131073, 262145, 2097152, 2097153])
@pytest.mark.parametrize("alone", [False, True])
def test_select_draws(api, vocab, alone):
    """Draws after four rejections, the second of them without mass, that cross
    in the first, a middle and the last slice of the vocabulary (one token
    where the vocabulary is one past whole slices): by each slice width, by
    workgroup 0 alone after it gave up, and past the slices' reach."""
    lg, p, q, toks, u = _four_rejected(vocab, 900 + vocab)
    sel = sampling.branch_select(p, toks, q, u)
    assert sel.accepted is None and sel.flags == sampling.FLAG_ZERO_RESIDUAL
    st = api.new_stats(1)
    dl, dt, dq = dev(lg), dev(toks), dev(q)
    api.sb_softmax_stats(dl[None], 1.0, st)
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    f = api.lib.sb_internal_select_branch
    f.restype = C.c_int32
    f.argtypes = api.lib.sb_select_branch.argtypes + [C.c_uint64] + [C.c_int32] * 3
    per = _slice_tokens(vocab)
    last = (vocab - 1) // per

    def select(*uniforms):
        out = torch.full((3,), -7, dtype=torch.int32, device="cuda")
        du = dev(np.asarray(uniforms, np.float32))
        assert f(vocab, dl.data_ptr(), st.data_ptr(), 1.0, 4, dt.data_ptr(), dq.data_ptr(), du.data_ptr(), out.data_ptr(),
                 ws.data_ptr(), ws.numel(), api._stream(), 100000, 0, int(alone), 0) == 0
        return out.cpu().tolist()

    # the test after the rejection without mass reads p~ as it was before it
    say(f"select draws vocab={vocab} third candidate alone={alone}")
    assert select(0.9, 0.9, 0.7, 0.9, 0.5) == [2, toks[2], sampling.FLAG_ZERO_RESIDUAL]
    for g in sorted({0, last // 2, last}):
        uf = _uniform_into(sel.p_tilde, g * per, min(vocab, (g + 1) * per))
        tr = []
        sampling.branch_select(p, toks, q, u, trace=tr)
        want = sampling.draw(sel.p_tilde, float(uf), tr, 4)
        assert want // per == g
        assert decision_margin(tr, np.append(u, uf)) > TIE
        say(f"select draws vocab={vocab} slice {g} of {last + 1} alone={alone}")
        assert select(*u, uf) == [-1, want, sampling.FLAG_ZERO_RESIDUAL]


def test_select_past_the_slices_time(api):
    """One workgroup does a vocabulary past the slices' reach; reading along it,
    three rejections and a draw over 2.1 million tokens take 2 ms (24 ms when a
    thread summed a stretch of its own)."""
    vocab = 2100001
    lg, p, q, toks, u = _all_rejected(vocab, 3, 1.0, 5)
    st = api.new_stats(1)
    dl, dt, dq, du = dev(lg), dev(toks), dev(q), dev(np.append(u, np.float32(0.5)).astype(np.float32))
    api.sb_softmax_stats(dl[None], 1.0, st)
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    out = torch.zeros(3, dtype=torch.int32, device="cuda")
    best = 1e9
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        api.sb_select_branch(dl, st, 1.0, dt, dq, du, out, ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    print(f"select at {vocab} tokens: {best:.2f} ms", flush=True)
    assert out[0].item() == -1
    assert best < 8.0


def test_walk_wait_is_short(api):
    """Where one workgroup's messages never come, the others stop waiting after
    0.2 ms each (at most once per workgroup: who gives up leaves), and workgroup
    0 alone ends the walk: a call delayed by other work on the chip is late by
    well under a millisecond, not by the tens it would be worth waiting."""
    vocab = 32000
    lg, p, q, toks, u = _all_rejected(vocab, 3, 1.0, 6)
    sel = sampling.branch_select(p, toks, q, u)
    uf = _uniform_into(sel.p_tilde, 0, vocab)
    st = api.new_stats(1)
    dl, dt, dq, du = dev(lg), dev(toks), dev(q), dev(np.append(u, uf).astype(np.float32))
    api.sb_softmax_stats(dl[None], 1.0, st)
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    out = torch.zeros(3, dtype=torch.int32, device="cuda")
    f = api.lib.sb_internal_select_branch
    f.restype = C.c_int32
    f.argtypes = api.lib.sb_select_branch.argtypes + [C.c_uint64] + [C.c_int32] * 3
    best = 1e9
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        assert f(vocab, dl.data_ptr(), st.data_ptr(), 1.0, 3, dt.data_ptr(), dq.data_ptr(), du.data_ptr(), out.data_ptr(),
                 ws.data_ptr(), ws.numel(), api._stream(), 0, 1, 2, 0) == 0
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
        assert out.cpu().tolist() == [-1, sampling.draw(sel.p_tilde, float(uf)), 0]
    print(f"selection with one workgroup gone: {best:.2f} ms", flush=True)
    assert best < 2.0


def test_walk_flags(api):
    vocab = 64
    parents = synth.branch_parents(2, 2)
    lg, q, toks, u = _walk_case(vocab, parents, 1.0, 0.5, 77)
    q[1, toks[1]] = 0.0   # a drafted token with q(x) = 0
    lg[3, 5] = np.nan      # a non-finite target row
    ref = sampling.accept_resample(toks, parents, lg, 1.0, q, u)
    st = api.new_stats(len(parents))
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    res_t = api.new_result()
    dl = dev(lg)
    api.sb_softmax_stats(dl, 1.0, st)
    api.sb_accept_resample(dev(toks), parents, dl, st, 1.0, dev(q), dev(u), res_t, ws)
    got = api.decode_result(res_t)
    assert got["flags"] & api.SB_FLAG_NONFINITE
    assert ref.flags & sampling.FLAG_NONFINITE
    assert (got["flags"] & api.SB_FLAG_QZERO) == (ref.flags & sampling.FLAG_QZERO)


def test_host_rejects_bad_tree(api):
    vocab = 32
    ws = torch.empty(api.sb_sample_workspace_bytes(vocab), dtype=torch.uint8, device="cuda")
    lg = torch.zeros((3, vocab), device="cuda")
    st = api.new_stats(3)
    with pytest.raises(api.SBError) as e:
        api.sb_accept_resample(torch.zeros(3, dtype=torch.int32, device="cuda"), [-1, 0, 2], lg,
                               st, 1.0, torch.zeros((3, vocab), device="cuda"),
                               torch.zeros(3, device="cuda"), api.new_result(), ws)
    assert e.value.code == 2

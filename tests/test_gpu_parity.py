"""GPU parity: the HIP library (through its C ABI) against the float64 oracle.

Small configurations are compared on every row; the full-size configurations
run in the bench's launch configuration and are compared on sampled rows, and
on properties that hold at any size for every row.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import bridge, coupling, routing, verify
from paper_2609_36601_amd import workloads
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def np_out(out):
    """Per-row outputs as numpy arrays (bf16 tensors widened to float32)."""
    return {k: (v.float() if v.dtype == torch.bfloat16 else v).cpu().numpy()
            for k, v in out.items() if isinstance(v, torch.Tensor)}


def f64(x):
    return x.float().cpu().numpy().astype(np.float64)


def run_and_compare(saki, s, t, eps, seed, row_offset=0, rows=None, grad=True, valid=None,
                    grad_dtype=torch.float32, target_sample=False):
    say(f"couple n={s.shape[0]} V={s.shape[1]} dtype={s.dtype} eps={eps} offset={row_offset} "
        f"target_sample={target_sample}")
    vm = None if valid is None else torch.as_tensor(valid, dtype=torch.uint8, device=DEV)
    out = saki.couple(s, t, eps, seed, row_offset, route=True,
                      grad_dtype=grad_dtype if grad else None, valid_mask=vm, grad_scale=1.0,
                      correction_target=saki.SAKI_TARGET_SAMPLE if target_sample else saki.SAKI_TARGET_MODE)
    torch.cuda.synchronize()
    o = np_out(out)
    rows = np.arange(s.shape[0]) if rows is None else np.asarray(rows)
    g = f64(out["grad"][torch.as_tensor(rows, device=DEV)]) if grad else None
    R = parity.compare_couple(o, f64(s[torch.as_tensor(rows, device=DEV)]),
                              f64(t[torch.as_tensor(rows, device=DEV)]), eps, seed, row_offset,
                              rows, grad=g, valid=valid, target_sample=target_sample)
    say(R.summary())
    R.check()
    return out, o, R


def test_tiny_all_rows(saki_lib):
    s, t = workloads.rows("tiny", 0, 256, device=DEV)
    run_and_compare(saki_lib, s, t, 0.1, workloads.coupling_seed("tiny"))


@pytest.mark.parametrize("eps", [0.05, 0.2])
def test_mid_all_rows(saki_lib, eps):
    """The mid configuration (4,096 rows, V = 32,000 bf16, with the gradient)
    against the oracle on every row, the oracle spread over worker processes."""
    s, t = workloads.rows("mid", 0, 4096, device=DEV)
    seed = workloads.coupling_seed("mid")
    say(f"mid all rows eps={eps}")
    out = saki_lib.couple(s, t, eps, seed, 0, route=True, grad_dtype=torch.float32, grad_scale=1.0)
    torch.cuda.synchronize()
    o = np_out(out)
    _row_properties(o, eps)
    rows = np.arange(4096)
    R = parity.compare_couple_pool(o, f64(s), f64(t), eps, seed, 0, rows, grad=f64(out["grad"]))
    say(f"mid eps={eps}: {R.summary()}")
    R.check()


def _row_properties(o, eps, grad=None):
    assert np.all(o["row_status"] == 0)
    lam = o["lambda"]
    assert np.all((lam >= 0) & (lam <= 1))
    interior = lam < 1
    assert np.all(np.abs(o["kl"][interior] - eps) <= 2e-5 * eps)
    assert np.all(o["kl"] <= eps * (1 + 2e-5))
    # Cor. 1 (Pinsker) and Prop. 1 (correction rate = TV, on average)
    assert np.all(o["kl"] >= 0)
    assert np.all(o["tv"] <= np.sqrt(o["kl"] / 2) * (1 + 1e-5) + 1e-7)
    n = len(lam)
    rate, mean_tv = o["corrected"].mean(), o["tv"].mean()
    assert abs(rate - mean_tv) < 6 * np.sqrt(mean_tv * (1 - mean_tv) / n) + 1e-3
    acc = o["corrected"] == 0
    assert np.array_equal(o["token"][acc], o["proposal"][acc])


def _spread_rows(rng, n_seq, seq_len, per_seq):
    """Rows spread over the sequences: each sequence's first and last position
    and per_seq - 2 others at random."""
    out = []
    for q in range(n_seq):
        lo = q * seq_len
        mid = rng.choice(np.arange(lo + 1, lo + seq_len - 1), per_seq - 2, replace=False)
        out.extend([lo, lo + seq_len - 1, *mid.tolist()])
    return np.unique(np.asarray(out))


def test_large_full_size(saki_lib):
    """The large workload at full size (65,536 rows, V = 151,936 bf16, coupling +
    routed loss + f32 gradient) in the benchmark's launch configuration, at each
    radius of the sweep: 512 seeded rows spread over the 64 sequences (first and
    last position of each, six others) plus every row whose decision margin is
    below 1e-6 compared with the oracle element by element (events, tokens,
    lambda, KL, TV, losses, gradient rows); the properties that hold at any
    size checked on every row."""
    cfg = workloads.CONFIGS["large"]
    n, V = cfg["rows"], cfg["V"]
    say(f"generate large {n}x{V}")
    s = torch.empty(n, V, dtype=torch.bfloat16, device=DEV)
    t = torch.empty_like(s)
    workloads.fill("large", s, t)
    seed = workloads.coupling_seed("large")
    rows0 = _spread_rows(np.random.default_rng(3), 64, 1024, 8)
    assert rows0.size == 512
    for eps in cfg["eps"]:
        out = saki_lib.couple(s, t, eps, seed, 0, route=True, grad_dtype=torch.float32, grad_scale=1.0)
        torch.cuda.synchronize()
        o = np_out(out)
        _row_properties(o, eps)
        # every gradient row sums to zero (sum_j (p_j - 1[j = hot]) = 0)
        assert out["grad"][:4096].double().sum(dim=1).abs().max().item() < 1e-3
        near = np.nonzero(o["margin"] < parity.MARGIN)[0]
        rows = np.unique(np.concatenate([rows0, near]))
        ii = torch.as_tensor(rows, device=DEV)
        say(f"large eps={eps}: oracle on {rows.size} rows ({near.size} with GPU margin < 1e-6)")
        R = parity.compare_couple_pool(o, f64(s[ii]), f64(t[ii]), eps, seed, 0, rows, grad=f64(out["grad"][ii]))
        say(f"large eps={eps}: {R.summary()}")
        R.check()
        del out
        torch.cuda.empty_cache()
    del s, t
    torch.cuda.empty_cache()


@pytest.mark.parametrize("eps", [0.05, 0.5])
def test_large_other_radii(saki_lib, eps):
    s, t = workloads.rows("large", 0, 2048, device=DEV)
    rows = np.array([0, 700, 1500, 2047])
    out, o, R = run_and_compare(saki_lib, s, t, eps, workloads.coupling_seed("large"), rows=rows)
    _row_properties(o, eps)


@pytest.mark.parametrize("variant", ["", "shared"])
def test_stream_chunk(saki_lib, variant):
    chunk = 5
    lo = 4096 * chunk
    s, t = workloads.rows("stream", lo, lo + 4096, device=DEV, variant=variant)
    rows = np.array([0, 1, 2000, 4095])
    out, o, R = run_and_compare(saki_lib, s, t, 0.02, workloads.coupling_seed("stream"),
                                row_offset=lo, rows=rows)
    _row_properties(o, 0.02)


def test_verify_blocks(saki_lib):
    k = 8
    n = 4096 * 2
    s, t = workloads.rows("verify", 0, n, device=DEV)
    draft = workloads.drafts(s)
    eps = 0.2
    seed = workloads.coupling_seed("verify")
    say(f"verify n={n} k={k}")
    out = saki_lib.spec_verify(s, t, k, draft, eps, seed)
    torch.cuda.synchronize()
    gpu = dict(accepted_len=out["accepted_len"].cpu().numpy(),
               correction=out["correction"].cpu().numpy(),
               per_pos=np_out(out["per_pos"]))
    blocks = np.array([0, 1, 2, 500, 1023])
    idx = np.concatenate([np.arange(b * k, (b + 1) * k) for b in blocks])
    ii = torch.as_tensor(idx, device=DEV)
    R = parity.compare_verify(gpu, f64(s[ii]), f64(t[ii]), k, draft[ii].cpu().numpy(), eps, seed, 0,
                              blocks)
    say(R.summary())
    R.check()
    al = gpu["accepted_len"]
    assert al.min() >= 0 and al.max() <= k
    assert np.all((gpu["correction"] >= 0) == (al < k))
    say(f"mean accepted length {al.mean():.3f}")


def test_verify_without_per_position_outputs(saki_lib):
    """Without per-position outputs, drafts whose u lies below min(1, pi(z) / p(z))
    (a lower bound of the accept probability for every lambda in [0, 1]) are
    accepted without the lambda search; results equal the full path's and the
    oracle's."""
    k = 8
    n = 4096 * 2
    s, t = workloads.rows("verify", 0, n, device=DEV)
    draft = workloads.drafts(s)
    eps, seed = 0.2, workloads.coupling_seed("verify")
    say(f"verify without per-position outputs n={n}")
    full = saki_lib.spec_verify(s, t, k, draft, eps, seed)
    lean = saki_lib.spec_verify(s, t, k, draft, eps, seed, per_pos=False)
    torch.cuda.synchronize()
    gpu = dict(accepted_len=lean["accepted_len"].cpu().numpy(), correction=lean["correction"].cpu().numpy())
    same = (gpu["accepted_len"] == full["accepted_len"].cpu().numpy()) & \
           (gpu["correction"] == full["correction"].cpu().numpy())
    diff = np.nonzero(~same)[0]
    say(f"blocks differing from the full path: {diff.size}")
    assert diff.size <= 2
    blocks = np.unique(np.concatenate([[0, 1, 2, 500, 1023], diff]))
    idx = np.concatenate([np.arange(b * k, (b + 1) * k) for b in blocks])
    ii = torch.as_tensor(idx, device=DEV)
    R = parity.compare_verify(gpu, f64(s[ii]), f64(t[ii]), k, draft[ii].cpu().numpy(), eps, seed, 0,
                              blocks)
    say(R.summary())
    R.check()
    # EOS through the shortcut: p = pi accepts every draft
    V = 300
    s2 = torch.randn(2 * 4, V, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    d2 = torch.tensor([3, 7, 5, 1, 2, 2, 2, 2], dtype=torch.int32, device=DEV)
    out = saki_lib.spec_verify(s2, s2.clone(), 4, d2, 0.1, 5, eos_id=7, per_pos=False)
    torch.cuda.synchronize()
    assert out["accepted_len"].cpu().tolist() == [2, 4] and out["correction"].cpu().tolist() == [-1, -1]


def test_verify_full_size(saki_lib):
    """The verify workload at full size (8,192 blocks of k = 8, V = 151,936
    bf16) in the configuration the benchmark times (accepted lengths and
    corrections only): 512 seeded blocks spread over the 256 sequences (the
    first or last block of each, and one other) plus every block with a GPU
    decision margin below 1e-6 at an evaluated position against the oracle,
    and the first-rejection structure on every block."""
    cfg = workloads.CONFIGS["verify"]
    k, n, V = cfg["k"], cfg["rows"], cfg["V"]
    nb = n // k
    say(f"generate verify {n}x{V}")
    s = torch.empty(n, V, dtype=torch.bfloat16, device=DEV)
    t = torch.empty_like(s)
    workloads.fill("verify", s, t)
    draft = workloads.drafts(s)
    eps, seed = 0.2, workloads.coupling_seed("verify")
    out = saki_lib.spec_verify(s, t, k, draft, eps, seed, per_pos=False)
    full = saki_lib.spec_verify(s, t, k, draft, eps, seed)
    torch.cuda.synchronize()
    gpu = dict(accepted_len=out["accepted_len"].cpu().numpy(), correction=out["correction"].cpu().numpy())
    al, co = gpu["accepted_len"], gpu["correction"]
    assert al.shape == (nb,) and al.min() >= 0 and al.max() <= k
    assert np.all((co >= 0) == (al < k)) and co.max() < V
    # blocks with a near-tie accept decision at an evaluated position (the
    # margins come from the call with per-position outputs)
    margin = full["per_pos"]["margin"].cpu().numpy().reshape(nb, k)
    near = np.nonzero(np.nanmin(np.where(np.isnan(margin), np.inf, margin), axis=1) < parity.MARGIN)[0]
    rng = np.random.default_rng(11)
    per_seq = 32
    blocks0 = []
    for q in range(nb // per_seq):
        lo = q * per_seq
        edge = lo if q % 2 == 0 else lo + per_seq - 1
        other = rng.integers(lo + 1, lo + per_seq - 1)
        blocks0.extend([edge, other])
    blocks = np.unique(np.concatenate([np.asarray(blocks0), near]))
    idx = np.concatenate([np.arange(b * k, (b + 1) * k) for b in blocks])
    ii = torch.as_tensor(idx, device=DEV)
    say(f"verify: oracle on {blocks.size} blocks ({near.size} with a GPU margin < 1e-6)")
    R = parity.compare_verify_pool(gpu, f64(s[ii]), f64(t[ii]), k, draft[ii].cpu().numpy(), eps, seed, 0,
                                   blocks)
    say(f"verify: {R.summary()}; mean accepted length {al.mean():.3f}")
    R.check()
    del s, t, draft, out, full
    torch.cuda.empty_cache()


def test_verify_edge_cases(saki_lib):
    k, V = 4, 300
    rng = torch.Generator(device=DEV).manual_seed(1)
    s = torch.randn(3 * k, V, generator=rng, device=DEV)
    t = s.clone()
    t[k:] = torch.randn(2 * k, V, generator=rng, device=DEV)
    draft = torch.tensor([3, 7, 5, 1] * 3, dtype=torch.int32, device=DEV)
    draft[2 * k + 1] = 1000  # out of range
    out = saki_lib.spec_verify(s, t, k, draft, 0.1, 5, eos_id=7)
    torch.cuda.synchronize()
    al, co = out["accepted_len"].cpu().tolist(), out["correction"].cpu().tolist()
    o = verify.verify_blocks(f64(s), f64(t), k, draft.cpu().numpy(), 0.1, 5, 0, 7)
    assert al == o["accepted_len"].tolist() and co == o["correction"].tolist()
    assert al[0] == 2 and co[0] == -1  # p = pi: accepted through the EOS at position 1
    st = out["per_pos"]["row_status"].cpu().tolist()
    assert st[0:4] == [0, 0, 3, 3]
    if al[2] == 1:
        assert st[9] == 2


@pytest.mark.parametrize("nb, k", [(1, 1), (1, 64), (32, 8), (33, 8), (64, 8), (150, 7), (600, 1)])
def test_verify_positions_evaluated_ahead(saki_lib, nb, k):
    """Batches on both sides of one and two workgroups per CU: positions behind
    a block's stop (a rejection, an accepted EOS, bad logits, a draft outside
    the vocabulary) are evaluated ahead or skipped, and leave no trace."""
    V, eos, eps, seed = 600, 7, 0.1, 21
    g = torch.Generator(device=DEV).manual_seed(100 * nb + k)
    n = nb * k
    s = torch.randn(n, V, generator=g, device=DEV)
    t = s + 0.5 * torch.randn(n, V, generator=g, device=DEV)
    draft = torch.multinomial(s.softmax(1), 1, generator=g).squeeze(1).to(torch.int32)
    draft[torch.rand(n, generator=g, device=DEV) < 0.05] = eos
    draft[torch.rand(n, generator=g, device=DEV) < 0.02] = V + 3
    s[torch.rand(n, generator=g, device=DEV) < 0.02, 5] = float("nan")
    say(f"verify ahead nb={nb} k={k}")
    out = saki_lib.spec_verify(s, t, k, draft, eps, seed, eos_id=eos)
    lean = saki_lib.spec_verify(s, t, k, draft, eps, seed, eos_id=eos, per_pos=False)
    torch.cuda.synchronize()
    pp = np_out(out["per_pos"])
    gpu = dict(accepted_len=out["accepted_len"].cpu().numpy(), correction=out["correction"].cpu().numpy(), per_pos=pp)
    R = parity.compare_verify(gpu, f64(s), f64(t), k, draft.cpu().numpy(), eps, seed, 0, np.arange(nb), eos_id=eos)
    say(R.summary())
    R.check()
    assert torch.equal(out["accepted_len"], lean["accepted_len"]) and torch.equal(out["correction"], lean["correction"])
    # the position a block stops at: its correction, its EOS draft, or a bad position
    al, st = gpu["accepted_len"], pp["row_status"].reshape(nb, k)
    d = draft.cpu().numpy().reshape(nb, k)
    for b in range(nb):
        stop = int(al[b])
        if stop > 0 and d[b, stop - 1] == eos:
            stop -= 1
        assert np.all(st[b, :stop] == 0) and np.all(st[b, stop + 1:] == 3), (b, stop, st[b])
    skipped = (st == 3).reshape(-1)
    assert np.all(pp["token"][skipped] == -1) and np.all(np.isnan(pp["lambda"][skipped]))
    assert np.array_equal(pp["proposal"], draft.cpu().numpy()) and np.all(pp["corrected"][skipped] == 0)


@pytest.mark.parametrize("nb, k", [(3, 1), (40, 8), (300, 5)])
@pytest.mark.parametrize("field", ["token", "proposal", "teacher_argmax"])
def test_verify_with_an_output_in_the_drafts_buffer(saki_lib, nb, k, field):
    """A per-position int32 output may be written over the draft: every other
    output, the proposals of skipped positions among them, is as with buffers of
    their own."""
    V, n = 700, nb * k
    g = torch.Generator(device=DEV).manual_seed(nb)
    s = padded(torch.randn(n, V, generator=g, device=DEV))
    t = padded(s + torch.randn(n, V, generator=g, device=DEV))
    draft, _ = saki_lib.sample(s, 6)
    draft[torch.rand(n, generator=g, device=DEV) < 0.02] = V + 3
    s[torch.rand(n, generator=g, device=DEV) < 0.02, 5] = float("nan")
    say(f"verify {field} in the draft's buffer nb={nb} k={k}")
    ref = saki_lib.spec_verify(s, t, k, draft, 0.1, 21)
    pp = saki_lib.alloc_couple_out(n, DEV)
    pp[field] = draft.clone()
    acc, corr = (torch.empty(nb, dtype=torch.int32, device=DEV) for _ in range(2))
    ws = torch.empty(256, dtype=torch.uint8, device=DEV)
    saki_lib.saki_spec_verify(s, t, k, pp[field], 0.1, 21, 0, -1, acc, corr, pp, ws)
    torch.cuda.synchronize()
    assert torch.equal(acc, ref["accepted_len"]) and torch.equal(corr, ref["correction"])
    assert torch.equal(pp["proposal"], draft)
    for key in pp:
        x, y = pp[key].contiguous(), ref["per_pos"][key].contiguous()
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), key


@pytest.mark.parametrize("nb", [64, 256])
def test_verify_of_blocks_that_stop_at_once(saki_lib, nb):
    """Blocks of eight whose first draft the teacher all but excludes: the
    positions behind it are dropped as soon as the rejection is certain, so the
    call takes little longer than one with the first positions alone: 1.05 / 1.2
    times for 64 / 256 blocks (1.7 times when they are evaluated to the end
    beside them)."""
    k, V, eps, seed = 8, 151936, 0.2, 33
    g = torch.Generator(device=DEV).manual_seed(nb)
    s, t = (saki_lib.alloc_rows(nb * k, V, torch.bfloat16, DEV) for _ in range(2))
    for b in range(0, nb * k, 128):
        x = 4.3 * torch.randn(min(128, nb * k - b), V, generator=g, device=DEV)
        s[b:b + 128] = x
        t[b:b + 128] = 0.6 * x + 2.4 * torch.randn(x.shape, generator=g, device=DEV)
    draft, _ = saki_lib.sample(s, seed + 1)
    at = draft.long()[:, None]
    t.scatter_(1, at, s.gather(1, at) - 40.0)
    say(f"verify blocks that stop at once: {nb}")
    ws = torch.empty(256, dtype=torch.uint8, device=DEV)

    def call(ss, tt, kk, d):
        acc, corr = (torch.empty(nb, dtype=torch.int32, device=DEV) for _ in range(2))
        run = lambda: saki_lib.saki_spec_verify(ss, tt, kk, d, eps, seed, 0, -1, acc, corr, None, ws)  # noqa: E731
        run()
        return _min_ms(run), acc.cpu().numpy(), corr.cpu().numpy()

    whole, acc, corr = call(s, t, k, draft)
    # position 0 of every block (other rows of the random streams: times only)
    first, _, _ = call(s[::k], t[::k], 1, draft[::k].contiguous())
    say(f"ms: {whole:.3f}, first positions alone {first:.3f}; stopped at 0: {(acc == 0).mean():.2f}")
    assert whole <= 1.4 * first, (whole, first)
    full = saki_lib.spec_verify(s, t, k, draft, eps, seed)
    assert np.array_equal(acc, full["accepted_len"].cpu().numpy()) and np.array_equal(corr, full["correction"].cpu().numpy())
    assert (acc == 0).mean() > 0.8


def test_verify_precision_of_small_batches(saki_lib):
    """lambda*, KL and TV of batches of at most one block per CU against 64 bits:
    2e-6 at every position, three times the largest error measured (6e-7, the
    rounding of float sums; a node 2% away from lambda* leaves up to 7e-6)."""
    g = torch.Generator(device=DEV).manual_seed(10)
    n, V, eps, nb = 1600, 5000, 0.2, 200
    rho = 0.2 + 0.79 * torch.rand(n, 1, generator=g, device=DEV)
    s = 4.3 * torch.randn(n, V, generator=g, device=DEV)
    t = rho * s + 3.0 * torch.sqrt(1 - rho ** 2) * torch.randn(n, V, generator=g, device=DEV)
    s, t = padded(s.to(torch.bfloat16)), padded(t.to(torch.bfloat16))
    draft, _ = saki_lib.sample(s, 3)
    say("verify precision")
    pp = {}
    for a in range(0, n, nb):
        o = saki_lib.spec_verify(s[a:a + nb], t[a:a + nb], 1, draft[a:a + nb], eps, 5, row_offset=a)["per_pos"]
        for key in ("lambda", "kl", "tv"):
            pp.setdefault(key, []).append(o[key].cpu().numpy())
    b = bridge.bridge_rows(f64(s), f64(t), eps)
    for key, ref in (("lambda", b["lam"]), ("kl", b["kl"]), ("tv", b["tv"])):
        err = np.abs(np.concatenate(pp[key]) / ref - 1.0)
        say(f"{key}: rms {np.sqrt(np.mean(err ** 2)):.1e} max {err.max():.1e}")
        assert err.max() < 2e-6, (key, np.argsort(-err)[:5], np.sort(-err)[:5])


def padded(x):
    """Copy of a [n, V] tensor in storage whose row pitch is a multiple of 16 bytes."""
    n, V = x.shape
    per = 16 // x.element_size()
    buf = torch.zeros(n, (V + per - 1) // per * per, dtype=x.dtype, device=x.device)
    buf[:, :V] = x
    return buf[:, :V]


def test_edge_vocab_sizes_and_special_rows(saki_lib):
    g = torch.Generator(device=DEV).manual_seed(7)
    for V in (1, 7, 8, 1000, 1025, 3000):
        n = 24
        s = padded((2 * torch.randn(n, V, generator=g, device=DEV)).to(torch.bfloat16))
        t = padded((2 * torch.randn(n, V, generator=g, device=DEV)).to(torch.bfloat16))
        t[3] = s[3]            # p = pi
        t[4] = s[4] + 2.0      # p = pi (exact shift in bf16 for these magnitudes? compare oracle anyway)
        if V > 1:
            s[5, V // 2] = float("inf")
            t[6, 0] = float("nan")
        for eps in (0.0, 0.3):
            valid = np.ones(n, np.uint8)
            valid[::5] = 0
            run_and_compare(saki_lib, s, t, eps, 99, row_offset=10, valid=valid)


@pytest.mark.parametrize("V", [16 * 1024, 17 * 1024 + 5, 256 * 1024, 256 * 1024 + 1])
def test_row_cache_boundaries(saki_lib, V):
    """bf16 rows of up to 256 chunks keep each wave's last four full chunks in
    LDS: every chunk cached (16 chunks), one chunk per wave past that plus a
    ragged tail, the largest cached row (256 chunks), and one entry more (the
    variant without the cache).  Coupling, loss and gradient against the
    oracle on every row; the verify kernel on the same rows, whose blocks
    stop at their first rejection."""
    g = torch.Generator(device=DEV).manual_seed(V)
    n = 8
    s = (3.0 * torch.randn(n, V, generator=g, device=DEV) / 0.7).to(torch.bfloat16)
    t = (0.7 * s.float() + 0.7 * 3.0 * torch.randn(n, V, generator=g, device=DEV)).to(torch.bfloat16)
    s, t = padded(s), padded(t)
    run_and_compare(saki_lib, s, t, 0.2, 4242, row_offset=3)
    k = 4
    draft = workloads.drafts(s)
    out = saki_lib.spec_verify(s, t, k, draft, 0.2, 4242, 3)
    torch.cuda.synchronize()
    gpu = dict(accepted_len=out["accepted_len"].cpu().numpy(),
               correction=out["correction"].cpu().numpy(),
               per_pos=np_out(out["per_pos"]))
    R = parity.compare_verify(gpu, f64(s), f64(t), k, draft.cpu().numpy(), 0.2, 4242, 3,
                              np.arange(n // k))
    say(R.summary())
    R.check()


def test_bf16_gradient_and_masks(saki_lib):
    """bf16 gradient rows against the oracle's gradient (2e-3 absolute plus the
    bf16 rounding, 2^-8 relative), with masked rows (exact zeros)."""
    s, t = workloads.rows("mid", 0, 64, device=DEV)
    valid = (np.arange(64) % 3 != 0).astype(np.uint8)
    out = saki_lib.couple(s, t, 0.2, 3, 0, route=True, grad_dtype=torch.bfloat16,
                          valid_mask=torch.as_tensor(valid, device=DEV), grad_scale=1.0)
    torch.cuda.synchronize()
    o = np_out(out)
    rows = np.arange(64)
    R = parity.compare_couple(o, f64(s), f64(t), 0.2, 3, 0, rows, grad=f64(out["grad"]), valid=valid,
                              grad_rtol=2.0 ** -8)
    say(R.summary())
    R.check()
    assert torch.all(out["grad"][torch.as_tensor(valid == 0, device=DEV)] == 0)


def test_loss_sum_and_scale(saki_lib):
    """Events exact except counted near-margin rows; the scaled loss sum
    against the routed objective (Eq. general_objective) evaluated by the
    oracle on the GPU's own events."""
    s, t = workloads.rows("tiny", 0, 256, device=DEV)
    valid = (np.arange(256) % 4 != 1).astype(np.uint8)
    scale = np.float32(1.0 / valid.sum())
    out = saki_lib.couple(s, t, 0.1, 11, 0, route=True, grad_dtype=torch.float32,
                          valid_mask=torch.as_tensor(valid, device=DEV), grad_scale=float(scale))
    torch.cuda.synchronize()
    o = np_out(out)
    S, T = f64(s), f64(t)
    R = parity.compare_couple(o, S, T, 0.1, 11, 0, np.arange(256), valid=valid, grad_scale=float(scale))
    say(R.summary())
    R.check()
    logp, logpi = bridge.log_softmax(S), bridge.log_softmax(T)
    idx = np.arange(256)
    y = o["token"].astype(np.int64)
    adv = logpi[idx, y] - logp[idx, y]
    rl, ls, _ = routing.route_rows(S, y, o["corrected"], o["target"], adv, valid, float(scale), want_grad=False)
    assert abs(o["loss_sum"][0] - ls) <= 1e-5 * np.abs(rl * float(scale)).sum()
    for i in range(256):
        tol = parity.loss_atol(o["corrected"][i], adv[i], logp[i, y[i]]) if valid[i] else 0.0
        assert parity.close(o["row_loss"][i], rl[i], atol=tol), i


def test_route_loss_standalone(saki_lib):
    s, t = workloads.rows("mid", 0, 128, device=DEV)
    ev = saki_lib.couple(s, t, 0.2, 21, 0)
    adv = (ev["logt_token"] - ev["logp_token"]).contiguous()
    valid = torch.as_tensor((np.arange(128) % 7 != 2).astype(np.uint8), device=DEV)
    out = saki_lib.route_loss(s, ev["token"], ev["corrected"], ev["teacher_argmax"], adv,
                              valid_mask=valid, grad_scale=1.0)
    torch.cuda.synchronize()
    rl, ls, grad = routing.route_rows(f64(s), ev["token"].cpu().numpy(), ev["corrected"].cpu().numpy(),
                                      ev["teacher_argmax"].cpu().numpy(), adv.double().cpu().numpy(),
                                      valid.cpu().numpy(), 1.0)
    assert np.all(parity.close(out["row_loss"].cpu().numpy(), rl, atol=1e-6))
    assert abs(out["loss_sum"].item() - ls) <= 1e-5 * np.abs(rl).sum()
    assert np.max(np.abs(out["grad"].cpu().numpy() - grad)) <= parity.GRAD_ATOL


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 7169, 8191, 8192, 8193, 20000])
def test_loss_sum_row_counts(saki_lib, n):
    """The sum of the row losses at row counts around its wave, its workgroup and
    its group of loads in flight.  The sum is in double: it differs from the sum
    of the returned row losses by their rounding to float, 2^-24 of each."""
    g = torch.Generator(device=DEV).manual_seed(n)
    s = torch.randn(n, 16, generator=g, device=DEV)
    token = torch.randint(0, 16, (n,), generator=g, device=DEV, dtype=torch.int32)
    corrected = (torch.rand(n, generator=g, device=DEV) < 0.3).to(torch.uint8)
    adv = torch.randn(n, generator=g, device=DEV)
    say(f"loss sum n={n}")
    first = None
    for _ in range(2):
        out = saki_lib.route_loss(s, token, corrected, token, adv, grad_scale=0.25)
        torch.cuda.synchronize()
        rl = 0.25 * out["row_loss"].double().cpu().numpy()
        got = out["loss_sum"].item()
        assert abs(got - rl.sum()) <= 2.0 ** -23 * np.abs(rl).sum()
        assert first is None or got == first
        first = got


@pytest.mark.parametrize("V", [36 * 1024, 37 * 1024 + 5, 151936])
def test_route_loss_row_cache(saki_lib, V):
    """bf16 rows keep each wave's last nine full chunks of s in LDS between the
    routed loss's two sweeps: every chunk cached (nine per wave), one chunk per
    wave past that plus a ragged tail, and the large vocabulary (36 of its 148
    full chunks cached).  Loss and gradient against the oracle on every row,
    with a masked row and a bf16 gradient."""
    g = torch.Generator(device=DEV).manual_seed(V)
    n = 12
    s = padded((3.0 * torch.randn(n, V, generator=g, device=DEV) / 0.7).to(torch.bfloat16))
    token = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    vstar = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    corrected = (torch.arange(n, device=DEV) % 3 == 0).to(torch.uint8)
    adv = torch.randn(n, generator=g, device=DEV).float()
    valid = torch.as_tensor((np.arange(n) != 4).astype(np.uint8), device=DEV)
    say(f"route_loss V={V}")
    rl, ls, grad = routing.route_rows(f64(s), token.cpu().numpy(), corrected.cpu().numpy(),
                                      vstar.cpu().numpy(), adv.double().cpu().numpy(), valid.cpu().numpy(), 1.0)
    for gd in (torch.float32, torch.bfloat16):
        out = saki_lib.route_loss(s, token, corrected, vstar, adv, valid_mask=valid, grad_scale=1.0,
                                  grad_dtype=gd)
        torch.cuda.synchronize()
        assert np.all(parity.close(out["row_loss"].cpu().numpy(), rl, atol=1e-6))
        assert abs(out["loss_sum"].item() - ls) <= 1e-5 * np.abs(rl).sum()
        tol = parity.GRAD_ATOL if gd == torch.float32 else parity.GRAD_ATOL + 2.0 ** -8 * np.abs(grad)
        assert np.all(np.abs(out["grad"].float().cpu().numpy() - grad) <= tol)


def test_route_loss_f32_ragged_and_bad_rows(saki_lib):
    """f32 rows of a ragged vocabulary (no row cache), with a supervised index
    outside [0, V) at a valid row and a non-finite logit (both: NaN loss and a
    NaN gradient row), and a masked row with an invalid index (loss 0, gradient
    row 0); the other rows against the oracle."""
    g = torch.Generator(device=DEV).manual_seed(5)
    n, V = 10, 3000
    s = padded(2.0 * torch.randn(n, V, generator=g, device=DEV))
    token = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    vstar = torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    corrected = (torch.arange(n, device=DEV) % 2 == 1).to(torch.uint8)
    adv = torch.randn(n, generator=g, device=DEV).float()
    valid = torch.ones(n, dtype=torch.uint8, device=DEV)
    good = np.ones(n, bool)
    token[2], corrected[2] = V, 0                  # index outside the row
    vstar[3], corrected[3], valid[3] = -1, 1, 0    # masked, invalid index
    s[5, 17] = float("inf")                        # non-finite logit
    good[[2, 3, 5]] = False
    out = saki_lib.route_loss(s, token, corrected, vstar, adv, valid_mask=valid, grad_scale=1.0)
    torch.cuda.synchronize()
    rl_g, gr_g = out["row_loss"].cpu().numpy(), out["grad"].cpu().numpy()
    for r in (2, 5):
        assert np.isnan(rl_g[r]) and np.isnan(gr_g[r]).all()
    assert rl_g[3] == 0 and np.all(gr_g[3] == 0)
    ii = np.nonzero(good)[0]
    it = torch.as_tensor(ii, device=DEV)
    rl, _, grad = routing.route_rows(f64(s[it]), token[it].cpu().numpy(), corrected[it].cpu().numpy(),
                                     vstar[it].cpu().numpy(), adv[it].double().cpu().numpy(), None, 1.0)
    assert np.all(parity.close(rl_g[ii], rl, atol=1e-6))
    assert np.max(np.abs(gr_g[ii] - grad)) <= parity.GRAD_ATOL


@pytest.mark.parametrize("n", [1, 511, 512, 513, 1024, 1537, 1600])
def test_row_counts_around_the_grid(saki_lib, n):
    """Row counts at one, two and three rows per workgroup (512 on 256 CUs): one
    row per workgroup without the counter, rows taken ahead, and the last rows
    taken when a workgroup is free.  Every row equals the same row of calls of
    100 rows bit for bit, and the oracle on a sample; some rows have bad logits."""
    V = 1100
    g = torch.Generator(device=DEV).manual_seed(n)
    s = padded((2 * torch.randn(n, V, generator=g, device=DEV)).to(torch.bfloat16))
    t = padded((0.8 * s.float() + torch.randn(n, V, generator=g, device=DEV)).to(torch.bfloat16))
    s[torch.rand(n, generator=g, device=DEV) < 0.05, 3] = float("nan")
    say(f"couple n={n}")
    kw = dict(route=True, grad_dtype=torch.float32, grad_scale=0.5)
    out = saki_lib.couple(s, t, 0.2, 9, 40, **kw)
    torch.cuda.synchronize()
    for a in range(0, n, 100):
        part = saki_lib.couple(s[a:a + 100], t[a:a + 100], 0.2, 9, 40 + a, **kw)
        for k in part:
            if k != "loss_sum":
                x, y = out[k][a:a + 100].contiguous(), part[k].contiguous()
                assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (k, a)
    rows = np.unique(np.r_[0, n - 1, np.random.default_rng(n).integers(0, n, 24)])
    ii = torch.as_tensor(rows, device=DEV)
    R = parity.compare_couple(np_out(out), f64(s[ii]), f64(t[ii]), 0.2, 9, 40, rows, grad_scale=0.5)
    say(R.summary())
    R.check()


def test_determinism_and_row_split_invariance(saki_lib):
    s, t = workloads.rows("mid", 0, 512, device=DEV)
    a = saki_lib.couple(s, t, 0.2, 5, 1000, route=True, grad_dtype=torch.float32)
    b = saki_lib.couple(s, t, 0.2, 5, 1000, route=True, grad_dtype=torch.float32)
    c1 = saki_lib.couple(s[:200].contiguous(), t[:200].contiguous(), 0.2, 5, 1000, route=True,
                         grad_dtype=torch.float32)
    c2 = saki_lib.couple(s[200:].contiguous(), t[200:].contiguous(), 0.2, 5, 1200, route=True,
                         grad_dtype=torch.float32)
    torch.cuda.synchronize()
    for k in ("lambda", "kl", "tv", "proposal", "token", "corrected", "accept_prob", "grad", "row_loss"):
        assert torch.equal(a[k], b[k]), k
        assert torch.equal(a[k][:200], c1[k]) and torch.equal(a[k][200:], c2[k]), k


def test_zero_rows_is_a_no_op(saki_lib):
    s = torch.empty(0, 64, dtype=torch.bfloat16, device=DEV)
    out = saki_lib.couple(s, s, 0.1, 1, 0, route=True, grad_dtype=torch.float32)
    torch.cuda.synchronize()
    assert out["lambda"].numel() == 0


def _collect(o, rows, store, idx):
    for key, v in o.items():
        if key in ("grad", "loss_sum"):
            continue
        if key not in store:
            store[key] = np.zeros(idx, dtype=v.dtype)
        store[key][rows] = v


@pytest.mark.parametrize("variant", ["", "shared"])
def test_stream_full_size(saki_lib, variant):
    """The long-rollout stress workload (262,144 rows of V = 151,936 bf16,
    eps 0.02) in its 64 chunks of 4,096 rows, each call with its row_offset:
    8 seeded rows of every chunk (its first and last row, six others) plus every
    row with a GPU margin below 1e-6 against the oracle (512 rows); the
    'shared' variant (teacher = the student base, spike moved) on 4 chunks,
    32 rows each.  The properties that hold at any size on every row."""
    cfg = workloads.CONFIGS["stream"]
    V, chunk = cfg["V"], cfg["chunk"]
    n_total = cfg["rows"]
    eps, seed = 0.02, workloads.coupling_seed("stream")
    chunks = range(n_total // chunk) if variant == "" else (0, 21, 42, 63)
    per_chunk = 8 if variant == "" else 32
    s = torch.empty(chunk, V, dtype=torch.bfloat16, device=DEV)
    t = torch.empty_like(s)
    rng = np.random.default_rng(17)
    store, S, T, G, rows_all = {}, [], [], [], []
    n_near = 0
    for c in chunks:
        lo = c * chunk
        workloads.fill("stream", s, t, lo=lo, variant=variant)
        out = saki_lib.couple(s, t, eps, seed, lo, route=True, grad_dtype=torch.float32, grad_scale=1.0)
        torch.cuda.synchronize()
        o = np_out(out)
        _row_properties(o, eps)
        near = np.nonzero(o["margin"] < parity.MARGIN)[0]
        n_near += near.size
        loc = np.unique(np.concatenate([[0, chunk - 1], rng.choice(np.arange(1, chunk - 1), per_chunk - 2,
                                                                    replace=False), near]))
        ii = torch.as_tensor(loc, device=DEV)
        _collect({k: v[loc] for k, v in o.items() if k not in ("grad", "loss_sum")}, lo + loc, store, n_total)
        S.append(f64(s[ii]))
        T.append(f64(t[ii]))
        G.append(f64(out["grad"][ii]))
        rows_all.append(lo + loc)
        del out
    rows = np.concatenate(rows_all)
    say(f"stream{'/' + variant if variant else ''}: oracle on {rows.size} rows of {len(chunks)} chunks "
        f"({n_near} with GPU margin < 1e-6)")
    R = parity.compare_couple_pool(store, np.concatenate(S), np.concatenate(T), eps, seed, 0, rows,
                                   grad=np.concatenate(G))
    say(f"stream{'/' + variant if variant else ''}: {R.summary()}")
    R.check()
    del s, t
    torch.cuda.empty_cache()


@pytest.mark.parametrize("eps", [1e-4, 1e-3, 5e-3])
def test_annealing_radii(saki_lib, eps):
    """Radii of the annealing schedule (eps from 0.02 down to 0 over the first
    50 steps, Sec. 4.1; App. "Limiting Cases"), where the lambda sweeps and
    the final sweep take their expm1 forms: every tiny row, 64 rows of the
    large workload, both with the gradient, against the oracle."""
    s, t = workloads.rows("tiny", 0, 256, device=DEV)
    out, o, R = run_and_compare(saki_lib, s, t, eps, workloads.coupling_seed("tiny"))
    _row_properties(o, eps)
    s, t = workloads.rows("large", 0, 64, device=DEV)
    out, o, R = run_and_compare(saki_lib, s, t, eps, workloads.coupling_seed("large"))
    _row_properties(o, eps)


def test_annealing_stream_chunk(saki_lib):
    """A chunk of the long-rollout workload at eps = 4e-4 (step 49 of the
    linear schedule from 0.02 to 0 over 50 steps): its rows have
    lambda (d_max - c) above 60 at some search nodes, so the expm1 sweeps take
    their shifted form.  64 rows plus every near-margin row against the oracle."""
    lo = 4096 * 5
    eps, seed = 4e-4, workloads.coupling_seed("stream")
    s, t = workloads.rows("stream", lo, lo + 4096, device=DEV)
    out = saki_lib.couple(s, t, eps, seed, lo, route=True, grad_dtype=torch.float32, grad_scale=1.0)
    torch.cuda.synchronize()
    o = np_out(out)
    _row_properties(o, eps)
    rng = np.random.default_rng(5)
    near = np.nonzero(o["margin"] < parity.MARGIN)[0]
    loc = np.unique(np.concatenate([[0, 4095], rng.choice(4096, 62, replace=False), near]))
    ii = torch.as_tensor(loc, device=DEV)
    say(f"stream chunk eps={eps}: oracle on {loc.size} rows ({near.size} near-margin)")
    R = parity.compare_couple_pool(o, f64(s[ii]), f64(t[ii]), eps, seed, lo, loc, grad=f64(out["grad"][ii]))
    say(R.summary())
    R.check()


def _wide_rows(V, n, s_special, t_special, noise, seed):
    """Rows of N(0, 1) student logits whose teacher equals the student plus
    N(0, noise^2), except at one entry per row where the student logit is
    s_special and the teacher logit t_special: d = t - s spans more than 100
    there, so lambda* (d_max - c) exceeds 60 at the radii below and q/p can
    exceed float's range."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    s = torch.randn(n, V, generator=g, device=DEV)
    t = s + noise * torch.randn(n, V, generator=g, device=DEV)
    j = torch.randint(0, V, (n,), generator=g, device=DEV)
    r = torch.arange(n, device=DEV)
    s[r, j] = s_special
    t[r, j] = t_special
    return padded(s.to(torch.bfloat16)), padded(t.to(torch.bfloat16))


@pytest.mark.parametrize("V,s_sp,t_sp,noise,eps", [
    (151936, -80.0, 40.0, 0.3, 1.0),    # lambda* ~ 0.7: shifted node sums
    (151936, -80.0, 40.0, 0.3, 20.0),   # q concentrated on the special entry: q/p ~ e^92
    (151936, -100.0, 30.0, 0.0, 5e-3),  # small radius with lambda* (d_max - c) > 60: shifted expm1 sums
    (4096, -100.0, 30.0, 0.0, 2e-3),
])
def test_wide_range_rows(saki_lib, V, s_sp, t_sp, noise, eps):
    """Rows whose d = t - s spans more than 100: the lambda sweeps take their
    shifted exponents (lambda (d_max - c) > 60), in the plain or the expm1
    form, and the final sweep the form for q/p beyond float's range.  Every
    row against the oracle, with the gradient."""
    s, t = _wide_rows(V, 8, s_sp, t_sp, noise, 1000 + V)
    out, o, R = run_and_compare(saki_lib, s, t, eps, 31337, row_offset=40)
    assert np.all(np.isfinite(o["tv"])) and np.all(o["row_status"] == 0)
    lam = o["lambda"]
    say(f"lambda* {np.round(lam, 4).tolist()}")
    assert np.all(lam < 1)


@pytest.mark.parametrize("sigma", [0.05, 0.01])
def test_endpoint_small_kl(saki_lib, sigma):
    """t = s + N(0, sigma^2): KL(pi || p) ~ sigma^2 / 2 lies below both the
    radius 0.02 and 0.01, so lambda* = 1 and the endpoint is resolved with the
    expm1 form of the sweep (and the final sweep's).  Every row against the
    oracle."""
    g = torch.Generator(device=DEV).manual_seed(int(sigma * 1000))
    n, V = 32, 3000
    s = 2.0 * torch.randn(n, V, generator=g, device=DEV)
    t = s + sigma * torch.randn(n, V, generator=g, device=DEV)
    s, t = padded(s), padded(t)
    out, o, R = run_and_compare(saki_lib, s, t, 0.02, 404)
    assert np.all(o["lambda"] == 1.0)
    assert np.all(o["kl"] < 0.01)


def _redo_rows(n, V, D, seed):
    """Rows whose TV is too small for the plain forms' rounding: five entries
    share max p ~ 0.2, and one entry with p ~ 1e-23 carries the whole KL of 0.2
    (t - s = D there), so TV ~ 0.0044 lies below 0.02 sqrt(max p)."""
    rng = np.random.default_rng(seed)
    s = np.full((n, V), -10.0) + rng.normal(0, 0.01, (n, V))
    s[:, :5] = rng.normal(0, 0.01, (n, 5))
    j = rng.integers(5, V, n)
    s[np.arange(n), j] = -50.0
    t = s.copy()
    t[np.arange(n), j] += D
    S = torch.as_tensor(s, dtype=torch.float32, device=DEV)
    T = torch.as_tensor(t, dtype=torch.float32, device=DEV)
    return padded(S), padded(T)


def _check_redo_rows(s, t):
    """The oracle confirms that the rows meet the condition of a second pass."""
    b = bridge.bridge_rows(f64(s), f64(t), 0.2)
    pmax = np.exp(b["logp"]).max(axis=1)
    assert np.all(b["kl"] >= 0.1) and np.all(pmax < 0.25) and np.all(b["tv"] < 0.02 * np.sqrt(pmax))


@pytest.mark.parametrize("D", [60.0, 70.0])
def test_rows_resolved_again_in_the_expm1_forms(saki_lib, D):
    """Rows that a workgroup resolves again, in place, with every sweep in the
    expm1 form.  Every row against the oracle, with the gradient."""
    S, T = _redo_rows(16, 3000, D, int(D))
    _check_redo_rows(S, T)
    out, o, R = run_and_compare(saki_lib, S, T, 0.2, 8080, row_offset=7)
    _row_properties(o, 0.2)


def _mixed_redo_rows(n, V, every, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    s = padded(2.0 * torch.randn(n, V, generator=g, device=DEV))
    t = padded(0.8 * s + torch.randn(n, V, generator=g, device=DEV))
    rows = np.unique(np.r_[0, 1, np.arange(0, n, every), n - 2, n - 1])
    ii = torch.as_tensor(rows, device=DEV)
    s[ii], t[ii] = _redo_rows(rows.size, V, 60.0, seed)
    _check_redo_rows(s[ii], t[ii])
    return s, t, rows


@pytest.mark.parametrize("n, every", [(1600, 7), (1600, 1), (600, 3)])
def test_rows_resolved_again_among_rows_from_the_counter(saki_lib, n, every):
    """The same rows spread over a batch of more rows than workgroups: a row is
    resolved again while the workgroup's next row has been taken already, and
    among the last two rows per workgroup, where none is taken ahead.  Every row
    is written, equals the row of a call of 100 rows (one per workgroup) bit for
    bit, and the resolved rows match the oracle."""
    V = 3000
    s, t, rows = _mixed_redo_rows(n, V, every, 3)
    say(f"couple rows resolved again n={n} every={every}")
    kw = dict(route=True, grad_dtype=torch.float32, grad_scale=0.5)
    out = saki_lib.alloc_couple_out(n, DEV)
    for v in out.values():
        v.fill_(77)
    grad = saki_lib.alloc_rows(n, V, torch.float32, DEV)
    grad.fill_(77)
    route = dict(grad_scale=0.5, grad=grad, row_loss=torch.full((n,), 77.0, device=DEV),
                 loss_sum=torch.zeros(1, dtype=torch.float64, device=DEV))
    ws = torch.empty(saki_lib.workspace_bytes(saki_lib.SAKI_OP_COUPLE, n, V), dtype=torch.uint8, device=DEV)
    saki_lib.saki_couple(s, t, 0.2, 9, 40, out, route, ws)
    torch.cuda.synchronize()
    got = dict(out, grad=grad, row_loss=route["row_loss"])
    for a in range(0, n, 100):
        part = saki_lib.couple(s[a:a + 100], t[a:a + 100], 0.2, 9, 40 + a, **kw)
        for key in part:
            if key != "loss_sum":
                x, y = got[key][a:a + 100].contiguous(), part[key].contiguous()
                assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (key, a)
    pick = rows if rows.size <= 64 else np.unique(np.r_[rows[:8], rows[-8:], rows[::rows.size // 40]])
    ii = torch.as_tensor(pick, device=DEV)
    R = parity.compare_couple(np_out(got), f64(s[ii]), f64(t[ii]), 0.2, 9, 40, pick, grad=f64(grad[ii]) * 2.0)
    say(R.summary())
    R.check()


@pytest.mark.parametrize("nb, k", [(16, 4), (120, 5), (400, 3)])
def test_positions_resolved_again(saki_lib, nb, k):
    """Verification's own second pass, at most one position per CU, at most one
    block per CU, and more: every evaluated position against the oracle."""
    s, t, rows = _mixed_redo_rows(nb * k, 3000, 2, 4)
    draft, _ = saki_lib.sample(s, 8)
    say(f"verify positions resolved again nb={nb} k={k}")
    out = saki_lib.spec_verify(s, t, k, draft, 0.2, 17)
    torch.cuda.synchronize()
    gpu = dict(accepted_len=out["accepted_len"].cpu().numpy(), correction=out["correction"].cpu().numpy(),
               per_pos=np_out(out["per_pos"]))
    R = parity.compare_verify(gpu, f64(s), f64(t), k, draft.cpu().numpy(), 0.2, 17, 0, np.arange(nb))
    say(R.summary())
    R.check()
    assert (gpu["per_pos"]["row_status"][rows] == 0).sum() > rows.size // 2


def _min_ms(run, reps=7):
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("offset", [-200.0, -60.0, 60.0, 200.0])
def test_teacher_logits_with_an_offset(saki_lib, offset):
    """A constant added to every teacher logit changes neither pi nor anything
    computed from it: the coupling and the verification of the shifted rows give
    the unshifted rows' results to rounding, and take about their time (a row
    that loses its middle node to the offset falls back to lambda sweeps, half
    as long again).  Logits are multiples of 2^-12 so that the sum is exact."""
    n, V, eps, seed, k = 1024, 100000, 0.2, 71, 8
    g = torch.Generator(device=DEV).manual_seed(2)
    s, t, t2 = (saki_lib.alloc_rows(n, V, torch.float32, DEV) for _ in range(3))
    for a in range(0, n, 128):
        x = torch.randn(128, V, generator=g, device=DEV) * 3.0
        y = 0.8 * x + 1.8 * torch.randn(128, V, generator=g, device=DEV)
        s[a:a + 128] = (x * 4096).round() / 4096
        t[a:a + 128] = (y * 4096).round() / 4096
    t2.copy_(t + offset)
    draft, _ = saki_lib.sample(s, seed + 1)
    say(f"teacher offset {offset}")
    res, times = [], []
    for tt in (t, t2):
        out = saki_lib.alloc_couple_out(n, DEV)
        ws = torch.empty(saki_lib.workspace_bytes(saki_lib.SAKI_OP_COUPLE, n, V), dtype=torch.uint8, device=DEV)
        couple = lambda: saki_lib.saki_couple(s, tt, eps, seed, 0, out, None, ws)  # noqa: E731
        acc, corr = (torch.empty(n // k, dtype=torch.int32, device=DEV) for _ in range(2))
        verify = lambda: saki_lib.saki_spec_verify(s, tt, k, draft, eps, seed, 0, -1, acc, corr, None, ws)  # noqa: E731
        couple(), verify()
        times.append((_min_ms(couple), _min_ms(verify)))
        res.append(dict({key: v.cpu().numpy() for key, v in out.items()}, n=acc.cpu().numpy()))
    a, b = res
    assert np.array_equal(a["proposal"], b["proposal"])
    same = (a["corrected"] == b["corrected"])
    assert np.all(same | (a["margin"] < parity.MARGIN))
    for key in ("lambda", "kl", "tv", "accept_prob"):
        assert np.all(parity.close(b[key], a[key], rtol=3e-6)), (key, parity.rel_err(b[key], a[key]))
    say(f"ms (couple, verify): {times}")
    for i in range(2):
        assert times[1][i] <= 1.25 * times[0][i], times
    assert np.mean(a["n"] == b["n"]) > 0.99


@pytest.mark.parametrize("of", ["student", "teacher", "both"])
@pytest.mark.parametrize("eps", [0.005, 0.2])
def test_masked_leading_chunks(saki_lib, of, eps):
    """Waves whose first chunks hold a mask value (-1e4) in s, t or both, so that
    every sum of the stats sweep is rescaled from there when the wave meets an
    ordinary chunk, and d = t - s spans 1e4 where only one is masked: all rows
    against the oracle."""
    g = torch.Generator(device=DEV).manual_seed(4)
    n, V = 8, 9 * 1024 + 100
    s = 2.0 * torch.randn(n, V, generator=g, device=DEV)
    t = 0.8 * s + torch.randn(n, V, generator=g, device=DEV)
    if of != "teacher":
        s[:, :4 * 1024] = -1e4
    if of != "student":
        t[:, :4 * 1024] = -1e4
    run_and_compare(saki_lib, padded(s), padded(t), eps, 15)

"""GPU parity tests: every call goes through the C ABI (ctypes binding) and is compared with the
CPU oracle on the same seeded inputs -- bit-exact for histogram, decompositions and slice table,
max relative error <= 2e-2 (bf16 weights) / 6e-2 (fp8 weights) for the FFN."""

import numpy as np
import pytest
import torch

import oracle
import test_parts
import workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
FFN_TOL = {"bf16": 2e-2, "fp8": 6e-2}        # the contract: max relative error per (slice, expert) group
# Regression guard beside the contract.  One rounding of h and one of y to bf16 (2^-9 relative each, on sums whose
# terms partly cancel) put the error of these kernels at 3e-3 .. 5e-3 of a group's largest output; a result that is
# still inside the contract but several times that is a defect (a dropped K step, a misplaced scale), not rounding.
FFN_GUARD = {"bf16": 1e-2, "fp8": 1.5e-2}


def check_ffn_error(err, dtype, what=""):
    say("   %s max relative error %.3g" % (what, err))
    assert err <= FFN_TOL[dtype], (what, err)
    assert err <= FFN_GUARD[dtype], ("inside the contract but far above what these kernels have measured", what, err)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def dev_bf16(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def host_bf16_bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def say(*a):
    print(*a, flush=True)


# ------------------------------------------------------------------------------ histogram
@pytest.mark.parametrize("name", ["tiny", "c2", "c3"])
def test_histogram_configs(lib, name):
    cfg = workloads.CONFIGS[name]
    say("histogram", name)
    ids = workloads.config_routing(cfg)
    traffic, counts = lib.moe_route_histogram(dev(ids), cfg.E)
    torch.cuda.synchronize()
    rt, rc = oracle.route_histogram(ids, cfg.E)
    assert np.array_equal(traffic.cpu().numpy(), rt)
    assert np.array_equal(counts.cpu().numpy(), rc)


@pytest.mark.parametrize("N,T,topk,E,L", [(3, 7, 3, 6, 1), (4, 1, 1, 4, 2), (8, 5000, 5, 64, 3), (2, 40001, 1, 4096, 1),
                                          (16, 0, 2, 16, 1), (5, 33, 2, 640, 4)])
def test_histogram_shapes_and_invalid_ids(lib, N, T, topk, E, L):
    say("histogram shapes", N, T, topk, E, L)
    rng = np.random.default_rng(N * 1000 + T)
    ids = rng.integers(-2, E + 2, size=(L, N, T, topk), dtype=np.int64).astype(np.int32)   # includes invalid ids
    traffic, counts = lib.moe_route_histogram(dev(ids), E)
    t_only, none = lib.moe_route_histogram(dev(ids), E, want_counts=False)
    torch.cuda.synchronize()
    assert none is None
    for l in range(L):
        rt, rc = oracle.route_histogram(ids[l], E)
        assert np.array_equal(traffic[l].cpu().numpy(), rt)
        assert np.array_equal(counts[l].cpu().numpy(), rc)
        assert np.array_equal(t_only[l].cpu().numpy(), rt)


def test_histogram_argument_errors(lib):
    ids = torch.zeros((2, 4, 1), dtype=torch.int32, device=DEV)
    with pytest.raises(lib.MoeError):
        lib.moe_route_histogram(ids, 3)                     # E % N != 0
    with pytest.raises(lib.MoeError):
        lib.moe_route_histogram(ids, 8192)                  # E too large


# ------------------------------------------------------------------------------ decompositions
def check_decomposition(lib, which, mats, kmax, zero_diag):
    B, N, _ = mats.shape
    fn = lib.moe_decompose_greedy if which == "greedy" else lib.moe_decompose_bvn
    sentinel_p, sentinel_d = 0xEE, -777
    out0 = {"perms": torch.full((B, kmax, N), sentinel_p, dtype=torch.uint8, device=DEV),
            "durations": torch.full((B, kmax), sentinel_d, dtype=torch.int32, device=DEV)}
    out = fn(dev(mats), kmax, zero_diag=zero_diag, want_hashes=True, out=out0)
    torch.cuda.synchronize()
    ref = oracle.decompose_batch(which, mats, kmax, zero_diag=zero_diag, nthreads=8)
    counts = out["counts"].cpu().numpy()
    assert np.array_equal(counts, ref["counts"]), (which, N, counts, ref["counts"])
    perms = out["perms"].cpu().numpy()
    dur = out["durations"].cpu().numpy()
    for b in range(B):
        c = counts[b]
        assert np.array_equal(perms[b, :c], ref["perms"][b, :c]), (which, N, b)
        assert np.array_equal(dur[b, :c], ref["durations"][b, :c]), (which, N, b)
        assert (perms[b, c:] == sentinel_p).all() and (dur[b, c:] == sentinel_d).all()    # untouched past count
    assert np.array_equal(out["residual"].cpu().numpy(), ref["residual"])
    assert np.array_equal(out["hashes"].cpu().numpy().view(np.uint64), ref["hashes"])
    if which == "bvn":
        assert np.array_equal(out["pad_total"].cpu().numpy(), ref["pad_total"])
    # count/hash-only mode gives the same hashes
    lean = fn(dev(mats), kmax, zero_diag=zero_diag, want_perms=False, want_residual=False, want_hashes=True)
    torch.cuda.synchronize()
    assert np.array_equal(lean["hashes"].cpu().numpy().view(np.uint64), ref["hashes"])
    assert np.array_equal(lean["counts"].cpu().numpy(), ref["counts"])


# (N <= 16, <= 32, <= 64 and > 64 take different code paths in the greedy kernel)
SHAPES = [(1, 1.0, 10), (2, 1.0, 3), (3, 0.7, 4), (5, 0.6, 2), (8, 1.0, 1000), (15, 0.9, 77), (16, 0.5, 30),
          (16, 1.0, 100000000), (17, 0.6, 50), (24, 0.4, 7), (32, 0.9, 3000), (33, 0.3, 5),
          (64, 1.0, 100000), (65, 0.4, 9), (100, 0.8, 3), (128, 0.6, 40000)]


@pytest.mark.parametrize("N,density,high", SHAPES)
@pytest.mark.parametrize("zero_diag", [False, True])
def test_greedy_random(lib, N, density, high, zero_diag):
    say("greedy random", N, density, high, zero_diag)
    mats = workloads.random_matrices(6, N, seed=900 + N, density=density, high=high)
    mats[1] = 0                                                       # an all-zero matrix in the batch
    for kmax in (3, 2 * N + 2):
        check_decomposition(lib, "greedy", mats, kmax, zero_diag)


@pytest.mark.parametrize("N,density,high", SHAPES)
@pytest.mark.parametrize("zero_diag", [False, True])
def test_bvn_random(lib, N, density, high, zero_diag):
    say("bvn random", N, density, high, zero_diag)
    nb = 6 if N <= 65 else 2
    mats = workloads.random_matrices(nb, N, seed=1900 + N, density=density, high=high)
    mats[1] = 0
    check_decomposition(lib, "bvn", mats, 5, zero_diag)
    check_decomposition(lib, "bvn", mats, oracle.bvn_bound(N) if N <= 65 else 600, zero_diag)


@pytest.mark.parametrize("N,kmax", [(5, 3), (7, 26), (8, 50), (13, 20), (16, 60), (65, 9)])
@pytest.mark.parametrize("which", ["greedy", "bvn"])
def test_decompose_tail_is_zero(lib, which, N, kmax):
    """Tensors that the binding makes are zero behind the last matching, whatever the memory held (odd sizes: heads and tails of the 16-byte
    stores), and where only one of them is the caller's, that one is untouched there."""
    mats = workloads.random_matrices(5, N, seed=N + kmax, density=0.3, high=40)
    mats[1] = 0
    fn = getattr(lib, "moe_decompose_" + which)
    junk = [torch.full((5 * kmax * N + n,), 0xA5, dtype=torch.uint8, device=DEV) for n in (0, 16 * 5 * kmax)]
    del junk                                                             # (its memory is what the call's tensors are made of)
    o = fn(dev(mats), kmax)
    mine = torch.full((5, kmax), -7, dtype=torch.int32, device=DEV)
    o2 = fn(dev(mats), kmax, out={"durations": mine})
    torch.cuda.synchronize()
    assert int(o["counts"][1]) == 0 and torch.equal(o["perms"], o2["perms"]) and torch.equal(o["counts"], o2["counts"])
    for b in range(5):
        c = int(o["counts"][b])
        assert not bool(o["perms"][b, c:].any()) and not bool(o["durations"][b, c:].any())
        assert bool((mine[b, c:] == -7).all()) and torch.equal(mine[b, :c], o["durations"][b, :c])


def test_decompose_special_cases(lib):
    say("decompose special cases")
    n = 16
    eye = np.zeros((3, n, n), dtype=np.int32)
    eye[0] = np.eye(n, dtype=np.int32)[np.random.default_rng(0).permutation(n)] * 7      # c * P
    eye[1] = 1                                                                            # all ones
    eye[2] = np.outer(np.arange(1, n + 1), np.arange(2, n + 2))                           # unique optimum
    for which in ("greedy", "bvn"):
        check_decomposition(lib, which, eye, 300, False)
        check_decomposition(lib, which, eye, 0, False)                                    # kmax = 0
    big = np.full((1, 8, 8), (1 << 28) - 1, dtype=np.int32)                               # N * max < 2^31
    check_decomposition(lib, "greedy", big, 20, False)
    check_decomposition(lib, "bvn", big, 100, False)
    with pytest.raises(lib.MoeError):
        lib.moe_decompose_greedy(torch.zeros((1, 129, 129), dtype=torch.int32, device=DEV), 4)


@pytest.mark.parametrize("N,limit", [(2, 21), (16, 21), (31, 21), (64, 21), (65, 20), (128, 20)])
def test_greedy_keys_of_32_bits(lib, N, limit):
    """The search packs distance and column into one key while the duals stay below 2^limit and keeps them apart beyond: entries
    just below, around and above half of that (max u + max v of the first matching is the largest entry), one row or column far
    above the rest, and a matrix whose later matchings fall below the limit again."""
    say("greedy keys of 32 bits", N, limit)
    rng = np.random.default_rng(N)
    mats = np.stack([rng.integers(h // 2, h, (N, N)) for h in (1 << (limit - 2), 1 << (limit - 1), (1 << limit) - 1, 1 << limit, 1 << (limit + 1))]
                    + [rng.integers(0, 50, (N, N)) for _ in range(4)]).astype(np.int32)
    mats[5, 0] += (1 << limit) - 60                                       # one row / column above the rest
    mats[6, :, N - 1] += (1 << limit) - 25
    mats[7, N // 2] += 1 << (limit + 2)
    mats[8, 0, 0] = (1 << 30) // N                                        # gone after the first matching
    for kmax in (4, 2 * N):
        check_decomposition(lib, "greedy", mats, kmax, False)


@pytest.mark.parametrize("N,high", [(16, 2000000), (33, 2000000), (64, 2000000), (96, 1000000), (128, 1000000)])
def test_greedy_keys_whose_bound_is_taken_again(lib, N, high):
    """Entries just below the largest that keys have room for: the duals stay below it, the sum of the lengths of a matching's searches, by which they
    are bounded between two looks at them, does not (128 ranks, uniform up to 10^6: 1.25 and 1.04 million)."""
    say("greedy keys whose bound is taken again", N, high)
    mats = np.random.default_rng(N).integers(0, high, (6, N, N)).astype(np.int32)
    for kmax in (4, N):
        check_decomposition(lib, "greedy", mats, kmax, False)


def test_greedy_16_bit_residual(lib):
    """How the residual is held on chip (32 bits, or 16 bits with a second launch for the matrices that do not fit)
    does not change a byte of the result."""
    say("greedy 16-bit residual")
    for N, kmax in ((5, 12), (16, 8), (64, 70), (128, 32)):
        mats = workloads.random_matrices(4, N, seed=70 + N, density=0.8, high=65536)
        mats[0, 0, 1 % N] = 65535
        mats[2, N - 1, 0] = 65536                                        # does not fit 16 bits: redone in 32
        mats[3] = mats[3] * 3                                            # most entries do not fit
        a = lib.moe_decompose_greedy(dev(mats), kmax, zero_diag=True, want_hashes=True, residual_bits=32)
        b = lib.moe_decompose_greedy(dev(mats), kmax, zero_diag=True, want_hashes=True, residual_bits=16)
        c = lib.moe_decompose_greedy(dev(mats), kmax, zero_diag=True, want_hashes=True)
        torch.cuda.synchronize()
        for key in ("perms", "durations", "counts", "residual", "hashes"):
            assert torch.equal(a[key], b[key]) and torch.equal(a[key], c[key]), (N, key)
        ref = oracle.decompose_batch("greedy", mats, kmax, zero_diag=True)
        assert np.array_equal(b["hashes"].cpu().numpy().view(np.uint64), ref["hashes"])
        assert np.array_equal(b["counts"].cpu().numpy(), ref["counts"])
    stress = workloads.stress_matrices(16, 128)
    assert stress.max() < 65536
    b = lib.moe_decompose_greedy(dev(stress), 32, zero_diag=True, want_hashes=True, residual_bits=16)
    torch.cuda.synchronize()
    ref = oracle.decompose_batch("greedy", stress, 32, zero_diag=True, nthreads=8)
    assert np.array_equal(b["hashes"].cpu().numpy().view(np.uint64), ref["hashes"])
    assert np.array_equal(b["residual"].cpu().numpy(), ref["residual"])


def test_decompose_profile_hook(lib):
    """The measurement hook records cycles, ticks and search steps per matrix and changes no result."""
    say("decompose profile hook")
    mats = workloads.random_matrices(5, 64, seed=9, density=0.8, high=5000)
    plain = lib.moe_decompose_greedy(dev(mats), 70, zero_diag=True, want_hashes=True)
    prof = torch.zeros((5, 4), dtype=torch.int64, device=DEV)
    lib.moe_decompose_profile(prof)
    try:
        timed = lib.moe_decompose_greedy(dev(mats), 70, zero_diag=True, want_hashes=True)
        torch.cuda.synchronize()
        p_greedy = prof.cpu().numpy().copy()
        lib.moe_decompose_bvn(dev(mats), 50, zero_diag=True)
        torch.cuda.synchronize()
        p_bvn = prof.cpu().numpy().copy()
    finally:
        lib.moe_decompose_profile(None)
    for key in ("perms", "durations", "counts", "residual", "hashes"):
        assert torch.equal(plain[key], timed[key]), key
    assert (p_greedy[:, 0] > 0).all() and (p_greedy[:, 1] > 0).all() and (p_greedy[:, 2] >= p_greedy[:, 3]).all() and (p_greedy[:, 3] > 0).all()
    clock_ghz = p_greedy[:, 0] / p_greedy[:, 1] * 0.1
    assert ((clock_ghz > 0.3) & (clock_ghz < 3.0)).all(), clock_ghz                 # cycles per 10 ns tick: a shader clock
    assert (p_bvn[:, 0] > 0).all() and (p_bvn[:, 2] == 0).all()
    before = prof.clone()
    lib.moe_decompose_greedy(dev(mats), 70, zero_diag=True)                       # recording is off again
    torch.cuda.synchronize()
    assert torch.equal(before, prof)


def test_mfma_probe(lib):
    """The measurement kernel runs, is timed under its name, and its accumulators hold what the loop defines: zero for
    zero operands; with varied operands every accumulator is the same product block added once per iteration, so
    twice the iterations give twice the value (up to fp32 rounding of the running sums)."""
    say("mfma probe")
    z = lib.moe_probe_mfma_bf16(0, 7, 3)
    torch.cuda.synchronize()
    assert z.shape == (3 * 256,) and bool((z == 0).all())
    lib.moe_kernel_timing_enable(True)
    a = lib.moe_probe_mfma_bf16(1, 8, 2).clone()
    b = lib.moe_probe_mfma_bf16(1, 16, 2).clone()
    torch.cuda.synchronize()
    lib.moe_kernel_timing_enable(False)
    kt = lib.moe_kernel_timing_read()
    assert kt["mfma_probe_kernel"][1] == 2 and kt["mfma_probe_kernel"][0] > 0
    assert bool(torch.isfinite(a).all()) and bool((a != 0).any())
    assert torch.allclose(b, 2 * a, rtol=1e-3, atol=1e-6)


def test_decompose_stress_matrices_128(lib):
    """The batched stress workload at its real shape (128 x 128, Zipf rows), a sample of matrices."""
    say("decompose stress 128")
    mats = workloads.stress_matrices(48, 128)
    check_decomposition(lib, "greedy", mats, 32, True)
    check_decomposition(lib, "bvn", mats[:8], 512, True)
    say("decompose stress 128: full BvN on 2 matrices")
    check_decomposition(lib, "bvn", mats[:2], oracle.bvn_bound(128), True)


def check_sinkhorn(lib, mats, kmax, zero_diag, sweeps, eps):
    """Bit-exact: both sides add in index order and divide in IEEE double precision."""
    B, N, _ = mats.shape
    out = lib.moe_decompose_sinkhorn_bvn(dev(mats), kmax, zero_diag=zero_diag, sweeps=sweeps, eps=eps)
    torch.cuda.synchronize()
    counts = out["counts"].cpu().numpy()
    perms, coef = out["perms"].cpu().numpy(), out["coeffs"].cpu().numpy()
    scaled, resid, devi = out["scaled"].cpu().numpy(), out["residual"].cpu().numpy(), out["deviation"].cpu().numpy()
    for b in range(B):
        rp, rc, rx, rr, rd = oracle.sinkhorn_bvn(mats[b], kmax=kmax, zero_diag=zero_diag, iters=sweeps, eps=eps)
        assert np.array_equal(scaled[b], rx), (N, b, np.abs(scaled[b] - rx).max())
        assert devi[b] == rd
        assert counts[b] == len(rp), (N, b, counts[b], len(rp))
        assert np.array_equal(perms[b, :len(rp)], rp), (N, b)
        assert np.array_equal(coef[b, :len(rp)], rc), (N, b)
        assert np.array_equal(resid[b], rr), (N, b)
        assert (coef[b, len(rp):] == 0).all()


@pytest.mark.parametrize("N,density,high", [(1, 1.0, 5), (2, 1.0, 3), (5, 0.7, 9), (8, 1.0, 1000), (16, 0.6, 300), (33, 0.5, 50),
                                            (64, 1.0, 5000), (65, 0.6, 20), (128, 0.7, 40000)])
@pytest.mark.parametrize("zero_diag", [False, True])
def test_sinkhorn_bvn_random(lib, N, density, high, zero_diag):
    say("sinkhorn bvn random", N, density, high, zero_diag)
    nb = 4 if N <= 65 else 2
    mats = workloads.random_matrices(nb, N, seed=2900 + N, density=density, high=high)
    mats[1] = 0
    check_sinkhorn(lib, mats, 4, zero_diag, sweeps=20, eps=1e-12)
    check_sinkhorn(lib, mats, min(N * N, 700), zero_diag, sweeps=60 if N <= 65 else 25, eps=1e-12)
    check_sinkhorn(lib, mats[:1], 10, zero_diag, sweeps=0, eps=0.5)              # no scaling at all: plain BvN steps on A


def test_sinkhorn_bvn_configs_and_errors(lib):
    say("sinkhorn bvn configs")
    for name in ("tiny", "c2", "c3"):
        cfg = workloads.CONFIGS[name]
        traffic, _ = oracle.route_histogram(workloads.config_routing(cfg), cfg.E)
        for zd in (False, True):
            check_sinkhorn(lib, traffic[None], oracle.bvn_bound(cfg.N), zd, sweeps=200, eps=1e-12)
    with pytest.raises(lib.MoeError):
        lib.moe_decompose_sinkhorn_bvn(torch.zeros((1, 4, 4), dtype=torch.int32, device=DEV), 4, sweeps=-1)
    with pytest.raises(lib.MoeError):
        lib.moe_decompose_sinkhorn_bvn(torch.zeros((1, 129, 129), dtype=torch.int32, device=DEV), 4)


# ------------------------------------------------------------------------------ slice table
@pytest.mark.parametrize("name,which", [("tiny", "greedy"), ("tiny", "bvn"), ("c2", "greedy"), ("c2", "bvn"), ("c3", "greedy")])
def test_slice_table(lib, name, which):
    say("slice table", name, which)
    cfg = workloads.CONFIGS[name]
    ids = workloads.config_routing(cfg)
    traffic, _ = oracle.route_histogram(ids, cfg.E)
    order = np.argsort(-traffic.sum(0), kind="stable")
    kmax = cfg.kmax if which == "greedy" else oracle.bvn_bound(cfg.N)
    d_ids, d_traffic = dev(ids), dev(traffic)
    fn = lib.moe_decompose_greedy if which == "greedy" else lib.moe_decompose_bvn
    sched = fn(d_traffic.unsqueeze(0), kmax, zero_diag=True)
    if which == "greedy":
        rp, rd, _ = oracle.decompose_greedy(traffic, kmax, zero_diag=True)
    else:
        rp, rd, _, _, _ = oracle.decompose_bvn(traffic, kmax, zero_diag=True)
    for r in (int(order[0]), int(order[len(order) // 2]), int(order[-1])):
        off = lib.moe_slice_table(d_ids, cfg.E, r, d_traffic, sched["perms"][0], sched["durations"][0], sched["counts"],
                                  kmax)
        torch.cuda.synchronize()
        ref, _ = oracle.slice_table(ids, cfg.E, r, traffic, rp, rd, kmax, want_rows=False)
        assert np.array_equal(off.cpu().numpy(), ref), (name, which, r)


def test_slice_table_many_windows(lib):
    """A hand-made schedule that wires one source to the receiver in thousands of matchings
    (more windows than fit in LDS) and ships one assignment at a time."""
    say("slice table many windows")
    N, E, T, topk, r = 4, 8, 6000, 1, 2
    rng = np.random.default_rng(3)
    ids = rng.integers(0, E, size=(N, T, topk)).astype(np.int32)
    traffic, _ = oracle.route_histogram(ids, E)
    kmax = 3000
    perms = np.tile(np.array([[r, 0, 1, 3]], dtype=np.uint8), (kmax, 1))      # source 0 -> r in every matching
    perms[::3] = np.array([1, r, 0, 3], dtype=np.uint8)                       # every third: source 1 -> r
    dur = rng.integers(0, 3, size=kmax).astype(np.int32)
    count = np.array([kmax - 5], dtype=np.int32)
    off = lib.moe_slice_table(dev(ids), E, r, dev(traffic), dev(perms), dev(dur), dev(count), kmax)
    torch.cuda.synchronize()
    ref, _ = oracle.slice_table(ids, E, r, traffic, perms[:kmax - 5], dur[:kmax - 5], kmax, want_rows=False)
    assert np.array_equal(off.cpu().numpy(), ref)


@pytest.mark.parametrize("name,which", [("tiny", "greedy"), ("tiny", "bvn"), ("c2", "greedy"), ("c2", "bvn"), ("c3", "greedy")])
def test_slice_table_rows(lib, name, which):
    """Row map: assignment index bit-exact with the oracle; the arrival index is the rank of that assignment among
    all assignments destined to r (sources in rank order, each in arrival order)."""
    say("slice table rows", name, which)
    cfg = workloads.CONFIGS[name]
    ids = workloads.config_routing(cfg)
    traffic, _ = oracle.route_histogram(ids, cfg.E)
    order = np.argsort(-traffic.sum(0), kind="stable")
    kmax = cfg.kmax if which == "greedy" else oracle.bvn_bound(cfg.N)
    d_ids, d_traffic = dev(ids), dev(traffic)
    if which == "greedy":
        rp, rd, _ = oracle.decompose_greedy(traffic, kmax, zero_diag=True)
    else:
        rp, rd, _, _, _ = oracle.decompose_bvn(traffic, kmax, zero_diag=True)
    pp = np.zeros((kmax, cfg.N), dtype=np.uint8)
    dd = np.zeros(kmax, dtype=np.int32)
    pp[:len(rp)], dd[:len(rd)] = rp, rd
    cnt = np.array([len(rp)], dtype=np.int32)
    for r in (int(order[0]), int(order[len(order) // 2]), int(order[-1])):
        M = int(traffic[:, r].sum())
        off, arr, asg = lib.moe_slice_table_rows(d_ids, cfg.E, r, d_traffic, dev(pp), dev(dd), dev(cnt), kmax, M)
        torch.cuda.synchronize()
        ref_off, ref_rows = oracle.slice_table(ids, cfg.E, r, traffic, rp, rd, kmax)
        assert np.array_equal(off.cpu().numpy(), ref_off), (name, which, r)
        assert np.array_equal(asg.cpu().numpy(), ref_rows), (name, which, r)
        assert np.array_equal(arr.cpu().numpy(), np.searchsorted(np.sort(ref_rows), ref_rows)), (name, which, r)
        only = lib.moe_slice_table_rows(d_ids, cfg.E, r, d_traffic, dev(pp), dev(dd), dev(cnt), kmax, M, want_assignment=False)
        torch.cuda.synchronize()
        assert only[2] is None and np.array_equal(only[1].cpu().numpy(), arr.cpu().numpy())


@pytest.mark.parametrize("T,topk", [(9001, 1), (8192, 1), (2731, 3), (5, 1), (20000, 2)])
def test_slice_table_walk_passes(lib, T, topk):
    """Assignments per source below, at and above what one pass of the walk covers, with ragged ends."""
    say("slice table walk passes T=%d topk=%d" % (T, topk))
    N, E, r = 5, 20, 3
    rng = np.random.default_rng(T + topk)
    ids = rng.integers(-2, E + 2, size=(N, T, topk)).astype(np.int32)
    traffic, _ = oracle.route_histogram(ids, E)
    kmax = 3
    rp, rd, _ = oracle.decompose_greedy(traffic, kmax, zero_diag=True)
    k = len(rd)
    perms = np.zeros((kmax, N), dtype=np.uint8); perms[:k] = rp
    dur = np.zeros(kmax, dtype=np.int32); dur[:k] = rd
    off = lib.moe_slice_table(dev(ids), E, r, dev(traffic), dev(perms), dev(dur), dev(np.array([k], dtype=np.int32)), kmax)
    torch.cuda.synchronize()
    ref, _ = oracle.slice_table(ids, E, r, traffic, rp, rd, kmax, want_rows=False)
    assert np.array_equal(off.cpu().numpy(), ref)


@pytest.mark.parametrize("T,topk,E", [(1, 1, 5), (255, 1, 20), (256, 1, 20), (257, 1, 320), (1365, 3, 20), (4096, 1, 20), (4097, 1, 20), (33000, 2, 20)])
def test_slice_table_rows_walk(lib, T, topk, E):
    """The row map's walk: assignments per source below, at and above a chunk (256) and a chunk of every wavefront (4096), all or
    few of them for the rank, 1 to 64 experts."""
    say("slice table rows walk", T, topk, E)
    N, r, kmax = 5, 3, 6
    rng = np.random.default_rng(T + E)
    ids = rng.integers(-2, E + 2, size=(N, T, topk)).astype(np.int32)
    ids[1] = r * (E // N)                                                       # one source sends everything to one expert of r
    traffic, _ = oracle.route_histogram(ids, E)
    rp, rd, _ = oracle.decompose_greedy(traffic, kmax, zero_diag=True)
    k = len(rd)
    perms = np.zeros((kmax, N), dtype=np.uint8); perms[:k] = rp
    dur = np.zeros(kmax, dtype=np.int32); dur[:k] = rd // 2                     # half of it is left over
    M = int(traffic[:, r].sum())
    off, arr, asg = lib.moe_slice_table_rows(dev(ids), E, r, dev(traffic), dev(perms), dev(dur), dev(np.array([k], dtype=np.int32)), kmax, M)
    torch.cuda.synchronize()
    ref_off, ref_rows = oracle.slice_table(ids, E, r, traffic, rp, rd // 2, kmax)
    assert np.array_equal(off.cpu().numpy(), ref_off) and np.array_equal(asg.cpu().numpy(), ref_rows)
    arrival = np.cumsum((ids.ravel() // (E // N) == r) & (ids.ravel() >= 0) & (ids.ravel() < E)) - 1
    assert np.array_equal(arr.cpu().numpy(), arrival[ref_rows])


def test_slice_table_rows_shapes_and_errors(lib):
    say("slice table rows shapes")
    rng = np.random.default_rng(8)
    # many experts per rank (64), ids outside [0, E) are dropped, a schedule that ships in small pieces
    N, E, T, topk, r = 3, 192, 700, 3, 1
    ids = rng.integers(-5, E + 5, size=(N, T, topk)).astype(np.int32)
    traffic, _ = oracle.route_histogram(ids, E)
    kmax = 40
    perms = np.tile(np.array([[1, 2, 0]], dtype=np.uint8), (kmax, 1))          # source 0 -> r
    perms[1::2] = np.array([2, 0, 1], dtype=np.uint8)                          # every other: source 2 -> r
    dur = rng.integers(0, 30, size=kmax).astype(np.int32)
    M = int(traffic[:, r].sum())
    off, arr, asg = lib.moe_slice_table_rows(dev(ids), E, r, dev(traffic), dev(perms), dev(dur), dev(np.array([kmax - 3], dtype=np.int32)), kmax, M)
    torch.cuda.synchronize()
    ref_off, ref_rows = oracle.slice_table(ids, E, r, traffic, perms[:kmax - 3], dur[:kmax - 3], kmax)
    assert np.array_equal(off.cpu().numpy(), ref_off) and np.array_equal(asg.cpu().numpy(), ref_rows)
    assert np.array_equal(np.sort(arr.cpu().numpy()), np.arange(M))
    # too many (window, expert) counters for the row map: refused, the plain table still works
    big_k = 8192 // 64 + 1
    with pytest.raises(lib.MoeError):
        lib.moe_slice_table_rows(dev(ids), E, r, dev(traffic), dev(np.zeros((big_k, N), dtype=np.uint8)),
                                 dev(np.zeros(big_k, dtype=np.int32)), dev(np.zeros(1, dtype=np.int32)), big_k, M)


# ------------------------------------------------------------------------------ FFN
def ffn_error(y_gpu_bits, y_ref, offsets, rows=None):
    """max over (slice, expert) groups of max|y - yref| / max|yref| on the given rows."""
    y = oracle.decode_bf16(y_gpu_bits)
    if rows is None:
        rows = np.arange(int(offsets[-1]))
    grp = np.searchsorted(offsets, rows, side="right") - 1
    worst, worst_elem = 0.0, 0.0
    for g in np.unique(grp):
        sel = grp == g
        scale = np.abs(y_ref[sel]).max()
        assert scale > 0
        diff = np.abs(y[sel] - y_ref[sel])
        worst = max(worst, float(diff.max() / scale))
        # (reported beside the contract's metric: element by element, with an absolute floor of 1e-3 of the group's
        #  largest value -- a plain elementwise ratio is meaningless next to zero)
        worst_elem = max(worst_elem, float((diff / np.maximum(np.abs(y_ref[sel]), 1e-3 * scale)).max()))
    say("   (elementwise |y - ref| / max(|ref|, 1e-3 max|ref|): %.3g)" % worst_elem)
    return worst


def upload_weights(W):
    if W.dtype == "bf16":
        return dict(w_gate=dev_bf16(W.w_gate), w_up=dev_bf16(W.w_up), w_down=dev_bf16(W.w_down))
    return dict(w_gate=dev(W.w_gate), w_up=dev(W.w_up), w_down=dev(W.w_down),
                s_gate=dev(W.s_gate), s_up=dev(W.s_up), s_down=dev(W.s_down))


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("tile_rows", ["64", "128", "256"])
@pytest.mark.parametrize("E_loc,d,f,M,S", [(1, 256, 512, 700, 3), (2, 512, 384, 1500, 4), (4, 256, 128, 333, 5)])
def test_ffn_small(lib, dtype, tile_rows, E_loc, d, f, M, S):
    say("ffn small", dtype, tile_rows, E_loc, d, f, M, S)
    lib.moe_ffn_tile_override(int(tile_rows))
    try:
        W = workloads.ffn_weights(E_loc, d, f, seed=d + f, dtype=dtype)
        x = workloads.activations(M + 9, d, seed=M)                                      # 9 spare rows past the last group
        offsets = workloads.random_offsets(S * E_loc, M, seed=M + S)
        y0 = torch.full((M + 9, d), 3.0, dtype=torch.bfloat16, device=DEV)
        y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, y=y0, **upload_weights(W))
        torch.cuda.synchronize()
        ref = oracle.expert_ffn_sliced(x, offsets, E_loc, W)
        yb = host_bf16_bits(y)
        check_ffn_error(ffn_error(yb[:M], ref, offsets), dtype)
        assert (oracle.decode_bf16(yb[M:]) == 3.0).all()                                  # rows past the end untouched
        # a row's result does not depend on how the rows are sliced: one slice per expert, same experts
        expert = (np.searchsorted(offsets, np.arange(M), side="right") - 1) % E_loc
        order = np.argsort(expert, kind="stable")
        off2 = np.zeros(E_loc + 1, dtype=np.int32)
        off2[1:] = np.cumsum(np.bincount(expert, minlength=E_loc))
        y2 = lib.moe_expert_ffn_sliced(dev_bf16(x[order]), dev(off2), 1, E_loc, **upload_weights(W))
        torch.cuda.synchronize()
        assert np.array_equal(host_bf16_bits(y2), yb[:M][order])
    finally:
        lib.moe_ffn_tile_override()


def test_ffn_buffers_at_addresses_with_bit_31_set(lib):
    """Output and workspace whose 64-bit addresses have bit 31 of the low word set (the kernels build buffer
    descriptors from the two halves of such addresses)."""
    say("ffn buffers above a 2 GiB boundary of the low address word")
    E_loc, d, f, M, S = 1, 256, 512, 700, 3
    W = workloads.ffn_weights(E_loc, d, f, seed=d + f)
    x = workloads.activations(M, d, seed=M)
    offsets = workloads.random_offsets(S * E_loc, M, seed=M + S)
    ws_bytes = lib.moe_ffn_workspace_bytes(M, d, f)
    y_bytes = M * d * 2
    pool = torch.empty(((1 << 32) + (64 << 20),), dtype=torch.uint8, device=DEV)
    low = pool.data_ptr() & 0xFFFFFFFF
    o = ((0x80000000 - low) % (1 << 32) + 255) // 256 * 256 + 4096
    o2 = (o + y_bytes + 255) // 256 * 256
    assert ((pool.data_ptr() + o) >> 31) & 1 and ((pool.data_ptr() + o2) >> 31) & 1 and o2 + ws_bytes <= pool.numel()
    y0 = pool[o:o + y_bytes].view(torch.bfloat16).view(M, d)
    ws = pool[o2:o2 + ws_bytes]
    for rows in ("256", "128"):
        lib.moe_ffn_tile_override(int(rows))
        try:
            y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, y=y0, workspace=ws, **upload_weights(W))
            torch.cuda.synchronize()
        finally:
            lib.moe_ffn_tile_override()
        check_ffn_error(ffn_error(host_bf16_bits(y), oracle.expert_ffn_sliced(x, offsets, E_loc, W), offsets), "bf16", "rows %s" % rows)
    del pool, y0, ws, y


def test_ffn_fp8_weights_expanded_once(lib):
    """Room in the workspace lets a call expand the fp8 weights to bf16, which rounds the scaled weights: the same result as without it, up to that
    rounding and the order of the fp32 sums."""
    say("ffn fp8: weights expanded to bf16 once per call")
    E_loc, d, f, M, S = 2, 256, 384, 4500, 3
    W = workloads.ffn_weights(E_loc, d, f, seed=77, dtype="fp8")
    x = workloads.activations(M, d, seed=78)
    offsets = workloads.random_offsets(S * E_loc, M, seed=79)
    up = upload_weights(W)
    base = lib.moe_ffn_workspace_bytes(M, d, f)
    extra = lib.moe_ffn_expanded_weights_bytes(E_loc, d, f)
    assert extra >= 3 * E_loc * d * f * 2
    ref = oracle.expert_ffn_sliced(x, offsets, E_loc, W)
    outs = []
    for nbytes in (base, base + extra):
        ws = torch.empty((nbytes,), dtype=torch.uint8, device=DEV)
        y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, workspace=ws, **up)
        torch.cuda.synchronize()
        yb = host_bf16_bits(y)
        check_ffn_error(ffn_error(yb, ref, offsets), "fp8", "workspace %d" % nbytes)
        outs.append(oracle.decode_bf16(yb))
    scale = np.abs(outs[0]).max()
    assert np.abs(outs[0] - outs[1]).max() <= 0.02 * scale


@pytest.mark.parametrize("E_loc,d,f,M,expanded", [(8, 512, 1408, 72000, True), (8, 512, 1408, 16383, False), (1, 2048, 1408, 4096, False), (2, 256, 384, 4500, False)])
def test_ffn_fp8_calls_that_expand(lib, E_loc, d, f, M, expanded):
    """fp8 weights are expanded where there is room, 2048 rows per expert and the fused kernel is the faster way all the same; a few thousand rows are
    worked on in tiles."""
    say("ffn fp8: calls that expand", E_loc, d, f, M)
    w = workloads.ffn_weights_on_device(E_loc, d, f, M, "fp8", DEV)
    x = workloads.activations_on_device(M, d, 83, DEV)
    off = (np.arange(E_loc + 1) * M // E_loc).astype(np.int32)
    base = lib.moe_ffn_workspace_bytes(M, d, f)
    for nbytes, want in ((base + lib.moe_ffn_expanded_weights_bytes(E_loc, d, f), expanded), (base, False)):
        if not want and nbytes > base and M < 2048 * E_loc:
            nbytes *= 2                                                   # (however much room there is)
        lib.moe_kernel_timing_enable(True)
        try:
            y = lib.moe_expert_ffn_sliced(x, dev(off), 1, E_loc, workspace=torch.empty((nbytes,), dtype=torch.uint8, device=DEV), **w)
            torch.cuda.synchronize()
            names = lib.moe_kernel_timing_read()
        finally:
            lib.moe_kernel_timing_enable(False)
        assert ("ffn_expand_fp8_kernel" in names) == want, names
        for e in range(E_loc):
            wg, wu, wd = float_weights(w, e)
            xs = x[off[e]:off[e] + 300].float()
            ref = (torch.nn.functional.silu(xs @ wg.t()) * (xs @ wu.t())) @ wd.t()
            check_ffn_error(float((y[off[e]:off[e] + 300].float() - ref).abs().max() / ref.abs().max()), "fp8", "expert %d" % e)


@pytest.mark.parametrize("mapped", [False, True])
def test_ffn_same_bits_every_run(lib, mapped):
    """Tiles are handed to workgroups dynamically, but the arithmetic of a tile is fixed: the output of a call
    must not change by a bit from run to run (a race inside the kernels would show here)."""
    say("ffn same bits every run", mapped)
    E_loc, d, f, S, M = 4, 1024, 768, 6, 21000
    W = workloads.ffn_weights(E_loc, d, f, seed=5, dtype="bf16")
    x = dev_bf16(workloads.activations(M, d, seed=6))
    offsets = dev(workloads.random_offsets(S * E_loc, M, seed=7))
    w = upload_weights(W)
    rng = np.random.default_rng(8)
    row_map = dev(rng.permutation(M).astype(np.int32))
    row_gate = dev(rng.random(M, dtype=np.float32))
    first = None
    for _ in range(6):
        if mapped:
            y = lib.moe_expert_ffn_sliced_mapped(x, offsets, S, E_loc, w["w_gate"], w["w_up"], w["w_down"], row_map, row_gate)
        else:
            y = lib.moe_expert_ffn_sliced(x, offsets, S, E_loc, **w)
        torch.cuda.synchronize()
        bits = y.view(torch.int16)
        if first is None:
            first = bits.clone()
        else:
            assert torch.equal(first, bits)


_MULTI = {}


def multi_tile_case(dtype):
    """36 000 rows in 6 x 4 ragged groups, d = 1536, f = 768: about 1000 tiles per phase, i.e. every workgroup runs
    several tiles and meets full blocks after full blocks, ragged ends of more and of fewer than 128 rows after either."""
    if dtype not in _MULTI:
        E_loc, d, f, S, M = 4, 1536, 768, 6, 36000
        W = workloads.ffn_weights(E_loc, d, f, seed=15, dtype=dtype)
        x = workloads.activations(M, d, seed=16)
        offsets = workloads.random_offsets(S * E_loc, M, seed=17)
        rng = np.random.default_rng(18)
        row_map = rng.permutation(M).astype(np.int32)
        gate = rng.uniform(0.05, 1.0, size=M).astype(np.float32)
        ref = oracle.expert_ffn_sliced(x, offsets, E_loc, W)
        ref_mapped, target = oracle.expert_ffn_sliced_mapped(x, offsets, E_loc, W, row_map, gate)
        _MULTI.clear()
        _MULTI[dtype] = dict(E_loc=E_loc, d=d, f=f, S=S, M=M, W=W, x=x, offsets=offsets, row_map=row_map, gate=gate, ref=ref,
                             ref_mapped=ref_mapped, target=target)
    return _MULTI[dtype]


@pytest.mark.parametrize("dtype,tile_rows,fixed", [("bf16", 0, 0), ("bf16", 0, 2), ("bf16", 256, 1), ("bf16", 128, 0), ("bf16", 64, 0),
                                                   ("fp8", 256, 0), ("fp8", 128, 0), ("fp8", 64, 0)])
def test_ffn_many_tiles_per_workgroup_all_rows(lib, dtype, tile_rows, fixed):
    """Every row against the oracle on a schedule large enough that the tile loop, the hand-over from one tile to the
    next (chained or not), ticket stealing, the counted-store wait and (both phases in one launch, the default for bf16
    weights and 256-row tiles) the wait of a phase-2 tile for its rows of h all run, for every kernel family
    (`fixed`: 0 = the call's own choice, 1 = tiles of 128 columns, 2 = adaptive-shape kernels, one launch per phase)."""
    say("ffn many tiles per workgroup", dtype, tile_rows, fixed)
    c = multi_tile_case(dtype)
    w = upload_weights(c["W"])
    sizes = np.diff(c["offsets"]) % 256
    assert ((sizes > 0) & (sizes <= 128)).any() and (sizes > 128).any() and (np.diff(c["offsets"]) >= 512).any()
    lib.moe_ffn_tile_override(tile_rows, fixed)
    try:
        x, off = dev_bf16(c["x"]), dev(c["offsets"])
        # (fp8: a workspace without room for expanded weights, so that the kernels that dequantise tile by tile run)
        ws = torch.empty((lib.moe_ffn_workspace_bytes(c["M"], c["d"], c["f"]),), dtype=torch.uint8, device=DEV)
        y = lib.moe_expert_ffn_sliced(x, off, c["S"], c["E_loc"], workspace=ws, **w)
        torch.cuda.synchronize()
        check_ffn_error(ffn_error(host_bf16_bits(y), c["ref"], c["offsets"]), dtype, "plain, all %d rows" % c["M"])
        y0 = torch.full((c["M"], c["d"]), 3.0, dtype=torch.bfloat16, device=DEV)
        ym = lib.moe_expert_ffn_sliced_mapped(x, off, c["S"], c["E_loc"], row_map=dev(c["row_map"]), row_gate=dev(c["gate"]),
                                              y=y0, workspace=ws, **w)
        torch.cuda.synchronize()
        check_ffn_error(ffn_error(host_bf16_bits(ym)[c["target"]], c["ref_mapped"], c["offsets"]), dtype, "mapped, all rows")
    finally:
        lib.moe_ffn_tile_override()


@pytest.mark.parametrize("tile_rows,fixed,panel", [(0, False, 1), (0, False, 2), (256, True, 2), (128, False, 1)])
def test_ffn_panel_walk_all_rows(lib, tile_rows, fixed, panel):
    """The tile walk in column panels (what a call chooses by itself only for experts whose weights outgrow the
    memory-side cache): 18 column units in 3 groups, walked 1 or 2 groups at a time; every row compared."""
    say("ffn panel walk", tile_rows, fixed, panel)
    E_loc, d, f, S, M = 2, 512, 2304, 3, 12000
    W = workloads.ffn_weights(E_loc, d, f, seed=25)
    x = workloads.activations(M, d, seed=26)
    offsets = workloads.random_offsets(S * E_loc, M, seed=27)
    lib.moe_ffn_tile_override(tile_rows, fixed, panel)
    try:
        y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, **upload_weights(W))
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    check_ffn_error(ffn_error(host_bf16_bits(y), oracle.expert_ffn_sliced(x, offsets, E_loc, W), offsets), "bf16", "all %d rows" % M)


@pytest.mark.parametrize("S,E_loc,tile_rows", [(375, 4, 0), (375, 4, 256), (1250, 4, 0), (1250, 4, 256), (5000, 1, 128)])
def test_ffn_thousands_of_groups_all_rows(lib, S, E_loc, tile_rows):
    """More (slice, expert) groups than the planning workgroup has threads (a full BvN schedule at 64 ranks has 3972
    slices): the plan is then built in several passes.  Ragged groups with empty ones; every row compared."""
    say("ffn thousands of groups", S, E_loc, tile_rows)
    d, f, M = 256, 256, 30000
    G = S * E_loc
    W = workloads.ffn_weights(E_loc, d, f, seed=G)
    x = workloads.activations(M + 3, d, seed=G + 1)
    offsets = workloads.random_offsets(G, M, seed=G + 2, empty_frac=0.3, power=12.0)     # a few groups of several tiles among crumbs
    assert (np.diff(offsets) == 0).sum() > G // 5 and (np.diff(offsets) > 256).any()
    lib.moe_ffn_tile_override(tile_rows)
    try:
        y0 = torch.full((M + 3, d), 3.0, dtype=torch.bfloat16, device=DEV)
        y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, y=y0, **upload_weights(W))
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    yb = host_bf16_bits(y)
    check_ffn_error(ffn_error(yb[:M], oracle.expert_ffn_sliced(x, offsets, E_loc, W), offsets), "bf16", "%d groups" % G)
    assert (oracle.decode_bf16(yb[M:]) == 3.0).all()


@pytest.mark.parametrize("tile_rows,fixed", [(0, False), (256, True), (64, False)])
def test_ffn_more_than_2_to_31_activation_elements(lib, tile_rows, fixed):
    """M * d just above 2^31 (rows are addressed with 64 bits): 8.4 M rows of 256 values in 3 x 2 groups, plain and
    through a row map; rows sampled from every group, whole tiles at the far end of the buffers included."""
    say("ffn M*d > 2^31", tile_rows, fixed)
    E_loc, d, f, S = 2, 256, 256, 3
    M = (1 << 31) // d + 4099
    assert M * d > (1 << 31)
    W = workloads.ffn_weights(E_loc, d, f, seed=41)
    w = upload_weights(W)
    offsets = workloads.random_offsets(S * E_loc, M, seed=42, empty_frac=0.0)
    x = workloads.activations_on_device(M, d, 43, DEV)
    rows = sample_rows(offsets, 300, blocks=[(M - 700, M), (offsets[3] - 300, offsets[3] + 300), (0, 256)])
    idx = torch.from_numpy(rows).to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(44)
    row_map = torch.randperm(M, device=DEV, generator=g).to(torch.int32)
    lib.moe_ffn_tile_override(tile_rows, fixed)
    try:
        y = lib.moe_expert_ffn_sliced(x, dev(offsets), S, E_loc, **w)
        torch.cuda.synchronize()
        ref = oracle.expert_ffn_sliced(_RowsView(host_bf16_bits(x[idx]), rows, M), offsets, E_loc, W, rows=rows)
        check_ffn_error(ffn_error(host_bf16_bits(y[idx]), ref, offsets, rows=rows), "bf16", "plain, %d sampled rows" % len(rows))
        del y
        ym = lib.moe_expert_ffn_sliced_mapped(x, dev(offsets), S, E_loc, row_map=row_map, **w)
        torch.cuda.synchronize()
        src = row_map[idx].long()                                        # arrival rows behind the sampled schedule rows
        ref = oracle.expert_ffn_sliced(_RowsView(host_bf16_bits(x[src]), rows, M), offsets, E_loc, W, rows=rows)
        check_ffn_error(ffn_error(host_bf16_bits(ym[src]), ref, offsets, rows=rows), "bf16", "mapped, %d sampled rows" % len(rows))
        del ym
    finally:
        lib.moe_ffn_tile_override()


def test_ffn_edge_cases(lib):
    say("ffn edge cases")
    E_loc, d, f = 2, 256, 128
    W = workloads.ffn_weights(E_loc, d, f, seed=1)
    up = upload_weights(W)
    x = workloads.activations(64, d, seed=2)
    # all groups empty: nothing is written
    y0 = torch.full((64, d), 5.0, dtype=torch.bfloat16, device=DEV)
    off = np.zeros(2 * E_loc + 1, dtype=np.int32)
    y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(off), 2, E_loc, y=y0, **up)
    torch.cuda.synchronize()
    assert (y.float() == 5.0).all()
    # a single row, and a group of exactly one tile plus one row
    for sizes in ([1, 0, 0, 0], [0, 0, 0, 1], [64, 0, 0, 0][::-1], [33, 31, 0, 0]):
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(off), 2, E_loc, **up)
        torch.cuda.synchronize()
        ref = oracle.expert_ffn_sliced(x, off, E_loc, W)
        check_ffn_error(ffn_error(host_bf16_bits(y)[:off[-1]], ref, off), "bf16", str(sizes))
    with pytest.raises(lib.MoeError):
        lib.moe_expert_ffn_sliced(dev_bf16(x[:, :128]), dev(off), 2, E_loc, w_gate=up["w_gate"][:, :, :128].contiguous(),
                                  w_up=up["w_up"][:, :, :128].contiguous(), w_down=up["w_down"][:, :128].contiguous())


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("tile_rows", ["64", "256"])
def test_ffn_mapped(lib, dtype, tile_rows):
    """Gather / scatter through a row map and the router weight in the epilogue."""
    say("ffn mapped", dtype, tile_rows)
    lib.moe_ffn_tile_override(int(tile_rows))
    try:
        E_loc, d, f, M, S = 2, 512, 384, 1500, 4
        rng = np.random.default_rng(77)
        W = workloads.ffn_weights(E_loc, d, f, seed=5, dtype=dtype)
        x = workloads.activations(M, d, seed=6)                                          # arrival order
        offsets = workloads.random_offsets(S * E_loc, M - 40, seed=7)                    # 40 arrival rows are never scheduled
        used = int(offsets[-1])
        row_map = rng.permutation(M)[:used].astype(np.int32)
        gate = rng.uniform(0.05, 1.0, size=used).astype(np.float32)
        y0 = torch.full((M, d), 3.0, dtype=torch.bfloat16, device=DEV)
        y = lib.moe_expert_ffn_sliced_mapped(dev_bf16(x), dev(offsets), S, E_loc, row_map=dev(row_map), row_gate=dev(gate),
                                             y=y0, **upload_weights(W))
        torch.cuda.synchronize()
        ref, target = oracle.expert_ffn_sliced_mapped(x, offsets, E_loc, W, row_map, gate)
        yb = host_bf16_bits(y)
        check_ffn_error(ffn_error(yb[target], ref, offsets), dtype)
        untouched = np.setdiff1d(np.arange(M), target)
        assert (oracle.decode_bf16(yb[untouched]) == 3.0).all()
        # identity map and unit gate: the very bytes of the plain call
        ident = np.arange(used, dtype=np.int32)
        ya = lib.moe_expert_ffn_sliced_mapped(dev_bf16(x), dev(offsets), S, E_loc, row_map=dev(ident),
                                              row_gate=dev(np.ones(used, dtype=np.float32)), **upload_weights(W))
        yp = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, **upload_weights(W))
        torch.cuda.synchronize()
        assert np.array_equal(host_bf16_bits(ya)[:used], host_bf16_bits(yp)[:used])
        # gathering through the map equals running the plain call on rows gathered beforehand
        yg = lib.moe_expert_ffn_sliced(dev_bf16(np.ascontiguousarray(x[row_map])), dev(offsets), S, E_loc, **upload_weights(W))
        ym = lib.moe_expert_ffn_sliced_mapped(dev_bf16(x), dev(offsets), S, E_loc, row_map=dev(row_map), **upload_weights(W))
        torch.cuda.synchronize()
        assert np.array_equal(host_bf16_bits(ym)[row_map], host_bf16_bits(yg)[:used])
    finally:
        lib.moe_ffn_tile_override()


@pytest.mark.parametrize("tile_rows", [0, 64, 256])
@pytest.mark.parametrize("S,E_loc,M", [(300, 4, 5000), (2, 3, 257), (9, 2, 513), (700, 2, 40), (2, 2050, 6000), (40, 1, 900)])
def test_ffn_slices_of_an_expert_share_tiles(lib, S, E_loc, M, tile_rows):
    """Rows are worked on expert by expert whatever their slice: a schedule of many slices gives the bits of the same rows
    sorted by expert in one slice (which needs no row list), plain and through a row map with weights.  Sizes: groups of a few
    rows, ends of row blocks, more groups than the planning workgroup has threads, more experts than it keeps in LDS."""
    say("ffn slices of an expert share tiles", S, E_loc, M, tile_rows)
    d, f = 256, 256
    g = torch.Generator(device=DEV)
    g.manual_seed(S + M)
    w = workloads.ffn_weights_on_device(E_loc, d, f, S, "bf16", DEV)
    offsets = workloads.random_offsets(S * E_loc, M, seed=S * E_loc, empty_frac=0.3)
    x = workloads.activations_on_device(M, d, M, DEV)
    expert = (np.searchsorted(offsets, np.arange(M), side="right") - 1) % E_loc
    order = dev(np.argsort(expert, kind="stable"))
    off1 = np.concatenate([[0], np.cumsum(np.bincount(expert, minlength=E_loc))]).astype(np.int32)
    row_map = torch.randperm(M, device=DEV, generator=g).to(torch.int32)
    gate = torch.rand((M,), device=DEV, generator=g)
    lib.moe_ffn_tile_override(tile_rows)
    try:
        y = lib.moe_expert_ffn_sliced(x, dev(offsets), S, E_loc, **w)
        want = lib.moe_expert_ffn_sliced(x[order].contiguous(), dev(off1), 1, E_loc, **w)
        ym = lib.moe_expert_ffn_sliced_mapped(x, dev(offsets), S, E_loc, row_map=row_map, row_gate=gate, **w)
        gathered = lib.moe_expert_ffn_sliced_mapped(x[row_map.long()].contiguous(), dev(offsets), S, E_loc,
                                                    row_map=torch.arange(M, dtype=torch.int32, device=DEV), row_gate=gate, **w)
        plain = lib.moe_expert_ffn_sliced(x[row_map.long()].contiguous(), dev(offsets), S, E_loc, **w)      # (by the same kernels)
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    assert torch.equal(y[order].view(torch.int16), want.view(torch.int16))
    assert torch.equal(ym[row_map.long()].view(torch.int16), gathered.view(torch.int16))
    # and the weighted rows are the plain ones times the weight, up to the two roundings to bf16 (2^-8 of the value each)
    plain = plain.float() * gate[:, None]
    assert bool(((gathered.float() - plain).abs() <= 2.0 ** -7 * plain.abs() + 1e-30).all())


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("E_loc,d,f,sizes", [
    (1, 256, 128, [[1]]), (1, 512, 1408, [[15]]), (2, 256, 384, [[16, 17]]), (1, 1280, 256, [[20], [0], [13], [30]]),
    (3, 256, 640, [[0, 65, 1], [64, 0, 0], [0, 0, 47]]), (2, 512, 128, [[3, 1]] * 300), (8, 4096, 256, [[9, 0, 33, 1, 64, 2, 0, 40]] * 2),
    (4, 256, 256, [[600, 3, 0, 80]]), (2, 8192, 128, [[129, 40]]), (1, 256, 4096, [[128]]), (1, 256, 4096, [[100], [29]]),
    (2, 2048, 384, [[166, 0], [30, 137]]), (1, 2048, 4096, [[200]]), (2, 512, 2048, [[1100, 0]]), (8, 256, 128, [[1100, 0, 0, 5, 0, 0, 0, 1]]),
    (2, 4096, 2048, [[81, 2]]), (1, 256, 128, [[17]]), (1, 512, 640, [[29]]), (2, 256, 256, [[18, 11]]), (6, 512, 1024, [[40, 0, 130, 33, 1, 9]]),
    (6, 512, 1024, [[100, 0, 0, 290, 1, 9]])])
def test_ffn_few_rows_per_expert(lib, dtype, E_loc, d, f, sizes):
    """The kernels that stream the weights: every row against the oracle, and through a row map with weights.  Sizes: ends of the
    16-row tiles and of the 64-row and 128-row chunks (128: the cases of one or two experts with f >= 2048 and of six), calls of up to 16 and up
    to 32 rows with their own kernels (32: up to 15, 17, 29 and 18 + 11 rows), more chunks than the grid has (1100 rows of one expert),
    experts without rows, more slices than a workgroup has threads, steps of K that do not divide by the wavefronts (2, 4, 6, 10, 20,
    22), x as it is and K-major (the 166 + 167 and the 200 rows of d = 2048), both strip widths of phase 2 (64 from E_loc * d / 64 >= half the
    compute units on: the 8 x 4096, 2 x 8192 and 2 x 4096 cases)."""
    say("ffn few rows per expert", dtype, E_loc, d, f, len(sizes))
    offsets = np.concatenate([[0], np.cumsum(np.array(sizes).ravel())]).astype(np.int32)
    M, S = int(offsets[-1]), len(sizes)
    W = workloads.ffn_weights(E_loc, d, f, seed=d + f, dtype=dtype)
    x = workloads.activations(M + 3, d, seed=M)
    w = upload_weights(W)
    y0 = torch.full((M + 3, d), 3.0, dtype=torch.bfloat16, device=DEV)
    y = lib.moe_expert_ffn_sliced(dev_bf16(x), dev(offsets), S, E_loc, y=y0, **w)
    torch.cuda.synchronize()
    ref = oracle.expert_ffn_sliced(x, offsets, E_loc, W)
    yb = host_bf16_bits(y)
    check_ffn_error(ffn_error(yb[:M], ref, offsets), dtype)
    assert (oracle.decode_bf16(yb[M:]) == 3.0).all()                                  # rows past the end untouched
    # row m at row_map[m], weighted: the same row products, so the plain result times the weight up to two roundings to bf16
    rng = np.random.default_rng(M)
    row_map, gate = rng.permutation(M).astype(np.int32), rng.random(M, dtype=np.float32)
    xm = np.empty_like(x[:M])
    xm[row_map] = x[:M]
    ones = lib.moe_expert_ffn_sliced_mapped(dev_bf16(xm), dev(offsets), S, E_loc, row_map=dev(row_map), **w)
    ym = lib.moe_expert_ffn_sliced_mapped(dev_bf16(xm), dev(offsets), S, E_loc, row_map=dev(row_map), row_gate=dev(gate), **w)
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16_bits(ones)[row_map], yb[:M])
    plain = oracle.decode_bf16(yb[:M]) * gate[:, None]
    assert (np.abs(oracle.decode_bf16(host_bf16_bits(ym)[row_map]) - plain) <= 2.0 ** -7 * np.abs(plain) + 1e-30).all()


@pytest.mark.parametrize("dtype,E_loc,d,f,M,S,streamed", [
    ("bf16", 1, 256, 512, 2048, 1, True), ("bf16", 1, 2048, 1408, 768, 3, True), ("bf16", 1, 2048, 1408, 4096, 1, False), ("fp8", 1, 4096, 1408, 768, 10, True),
    ("bf16", 8, 2048, 1408, 8 * 192, 10, True), ("bf16", 8, 2048, 1408, 8 * 256, 10, False), ("bf16", 16, 256, 256, 4096, 2, False), ("fp8", 64, 256, 256, 8192, 10, False),
    ("bf16", 64, 1024, 512, 512, 1, False), ("bf16", 64, 1024, 512, 256, 1, True), ("fp8", 64, 1024, 512, 2048, 1, True), ("fp8", 64, 1024, 512, 4096, 1, False),
    ("bf16", 2, 256, 256, 30, 1025, False)])
def test_ffn_choice_of_kernels(lib, dtype, E_loc, d, f, M, S, streamed):
    """Which calls stream the weights and which work in tiles (these run the planning kernel): many experts and a skewed spread of the
    rows must not meet the streaming kernels' re-reading of the weights.  Both ways agree where all rows belong to one expert."""
    say("ffn choice of kernels", dtype, E_loc, d, f, M, S)
    w = workloads.ffn_weights_on_device(E_loc, d, f, M, dtype, DEV)
    x = workloads.activations_on_device(M, d, S, DEV)
    sizes = np.zeros((S, E_loc), dtype=np.int64)
    sizes[:, E_loc // 2] = M // S
    sizes[0, E_loc // 2] += M - sizes.sum()
    offsets = dev(np.concatenate([[0], np.cumsum(sizes.ravel())]).astype(np.int32))
    lib.moe_kernel_timing_enable(True)
    try:
        y = lib.moe_expert_ffn_sliced(x, offsets, S, E_loc, **w)
        torch.cuda.synchronize()
        names = lib.moe_kernel_timing_read()
    finally:
        lib.moe_kernel_timing_enable(False)
    assert ("ffn_plan_kernel" not in names) == streamed
    lib.moe_ffn_tile_override(128)
    try:
        tiles = lib.moe_expert_ffn_sliced(x, offsets, S, E_loc, **w)
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    # the same values, h and y rounded to bf16 after sums in another order: single roundings of either differ
    assert float((y.float() - tiles.float()).norm() / tiles.float().norm()) <= 2.0 ** -8


def float_weights(w, e):
    """w_gate, w_up, w_down of expert e in float32."""
    out = []
    for k in ("gate", "up", "down"):
        v = w["w_" + k][e]
        if "s_" + k in w:
            v = v.view(torch.float8_e4m3fn).float() * w["s_" + k][e].repeat_interleave(128, 0).repeat_interleave(128, 1)
        out.append(v.float())
    return out


def check_against_float(x, off, y, w, what):
    """y of groups of one slice against float32 products on the GPU: two roundings to bf16 (hidden activations, result) of 2^-9 each at most."""
    for e in range(len(off) - 1):
        lo, hi = int(off[e]), int(off[e + 1])
        if lo == hi:
            continue
        wg, wu, wd = float_weights(w, e)
        xs = x[lo:hi].float()
        ref = (torch.nn.functional.silu(xs @ wg.t()) * (xs @ wu.t())) @ wd.t()
        diff = (y[lo:hi].float() - ref).abs()
        check_ffn_error(float(diff.max() / ref.abs().max()), "bf16", "%s expert %d" % (what, e))
        assert float(diff.norm() / ref.norm()) <= 2.0 ** -8, (what, e)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("E_loc,d,f,sizes,streamed", [
    (8, 1024, 512, [0, 0, 0, 1, 0, 0, 0, 0], True), (8, 1024, 512, [3, 0, 9, 0, 0, 1, 0, 3], True), (8, 1024, 512, [17, 0, 0, 0, 0, 0, 0, 0], True),
    (8, 1280, 640, [1, 0, 16, 0, 2, 0, 0, 13], True), (8, 1024, 512, [30, 0, 0, 2, 0, 0, 0, 1], None), (4, 2048, 384, [0, 2, 0, 0], True),
    (1, 7168, 256, [1], False), (1, 7168, 256, [32], False), (1, 7168, 256, [33], None)])
def test_ffn_up_to_32_rows(lib, dtype, E_loc, d, f, sizes, streamed):
    """Calls of up to 32 rows: which ones stream the weights, and strips of 16 weight rows where the experts that can hold rows have
    few strips (1 .. 32 rows of 8 x 1024, 8 x 1280 and 4 x 2048; 64 weight rows again at 33)."""
    say("ffn up to 32 rows", dtype, E_loc, d, f, sizes)
    M = sum(sizes)
    w = workloads.ffn_weights_on_device(E_loc, d, f, M, dtype, DEV)
    x = workloads.activations_on_device(M, d, M, DEV)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    lib.moe_kernel_timing_enable(True)
    try:
        y = lib.moe_expert_ffn_sliced(x, dev(off), 1, E_loc, **w)
        torch.cuda.synchronize()
        names = lib.moe_kernel_timing_read()
    finally:
        lib.moe_kernel_timing_enable(False)
    if streamed is not None:
        assert (not any("plan" in n for n in names)) == streamed
    check_against_float(x, off, y, w, "up to 32 rows")



@pytest.mark.parametrize("tile_rows,E_loc,d,f,sizes", [(0, 8, 1024, 512, [17, 0, 3, 0, 0, 1, 0, 0]), (0, 8, 1024, 512, [3, 0, 9, 0, 0, 1, 0, 3]),
                                                       (64, 2, 1024, 512, [70, 130]), (128, 2, 512, 1664, [140, 0])])
def test_ffn_fp8_large_activations(lib, tile_rows, E_loc, d, f, sizes):
    """Sums of 128 products with codes stay finite where y does, though the scale multiplies them only afterwards: x times 2^118 with the scales of the gate
    divided by it gives y times 2^118, bit by bit (scales are powers of two; no value leaves the normal range but the gate's scales, which stay exact)."""
    say("ffn fp8 large activations", tile_rows, E_loc, d, f, sizes)
    M, big = sum(sizes), 2.0 ** 118
    w = workloads.ffn_weights_on_device(E_loc, d, f, M, "fp8", DEV)
    for k in ("gate", "up", "down"):
        w["s_" + k] = torch.full_like(w["s_" + k], 2.0 ** -12)
    x = workloads.activations_on_device(M, d, M, DEV)
    off = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    lib.moe_ffn_tile_override(tile_rows)
    try:
        y = lib.moe_expert_ffn_sliced(x, off, 1, E_loc, **w)
        w["s_gate"] = torch.full_like(w["s_gate"], 2.0 ** -130)
        large = lib.moe_expert_ffn_sliced((x.float() * big).bfloat16(), off, 1, E_loc, **w)
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    assert bool(torch.isfinite(large).all()) and float(y.abs().max()) * big * 2 ** 12 > torch.finfo(torch.float32).max
    assert torch.equal(large, (y.float() * big).bfloat16())


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("tile_rows,kernels", [(64, 0), (128, 0), (256, 1)])
@pytest.mark.parametrize("d,f,sizes", [
    (256, 128, [1, 64, 65, 0, 31, 33]),                                   # contractions of one and two blocks of 128 values: no steady state
    (512, 384, [128, 129, 257, 63]),                                      # of three and four; row blocks and their remainders
    (2048, 1664, [70, 3]), (1536, 2048, [300]),                           # contractions split over workgroups: with a block more for some, in one phase only
    (3328, 256, [5, 40, 0, 1]),
    (1280, 640, [3500, 0, 70]), (256, 1152, [3137, 65])])                # many row blocks, walked for 8 column tiles at a time: 8 and 2, 8 and 8 and 2, or the only 2
def test_ffn_tile_edges(lib, dtype, tile_rows, kernels, d, f, sizes):
    """Tiles of 64, 128 and 256 rows: short contractions, remainders of rows, split contractions (the same bits on every call, which
    needs every counter of finished parts to start at zero and the parts to be added in order), and the same calls in a workspace without room for
    the parts' sums, which leaves them whole."""
    say("ffn tile edges", dtype, tile_rows, d, f, sizes)
    E_loc, M = len(sizes), sum(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    w = workloads.ffn_weights_on_device(E_loc, d, f, M + d, dtype, DEV)
    x = workloads.activations_on_device(M, d, M + f, DEV)
    need = lib.moe_ffn_workspace_bytes(M, d, f)
    least = need - (0 if max(d, f) < 1536 else 512 * 128 * 128 * 4)
    lib.moe_ffn_tile_override(tile_rows, kernels)
    try:
        ys = [lib.moe_expert_ffn_sliced(x, dev(off), 1, E_loc, y=torch.full_like(x, 9.0), workspace=torch.full((n,), 255, dtype=torch.uint8, device=DEV), **w)
              for n in (need, need, least)]
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    assert torch.equal(ys[0], ys[1])
    check_against_float(x, off, ys[0], w, "tiles")
    check_against_float(x, off, ys[2], w, "tiles, whole contractions")


@pytest.mark.parametrize("dtype,tile_rows,kernels", [("fp8", 0, 0), ("bf16", 64, 0), ("bf16", 128, 0), ("bf16", 256, 1)])
def test_ffn_tile_rows_addressed_with_64_bits(lib, dtype, tile_rows, kernels):
    say("ffn tiles, x above 4 GiB", dtype, tile_rows)
    d, f = 8192, 256
    M = (1 << 32) // (2 * d) + 700
    off = np.array([0, M - 1000, M], dtype=np.int32)
    w = workloads.ffn_weights_on_device(2, d, f, 71, dtype, DEV)
    x = workloads.activations_on_device(M, d, 72, DEV)
    lib.moe_ffn_tile_override(tile_rows, kernels)
    try:
        y = lib.moe_expert_ffn_sliced(x, dev(off), 1, 2, **w)
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    for lo, hi, e in ((0, 300, 0), (M - 1300, M - 1000, 0), (M - 1000, M, 1)):
        part = {k: v[e:e + 1] for k, v in w.items()}
        check_against_float(x[lo:hi], [0, hi - lo], y[lo:hi], part, "rows %d .." % lo)


@pytest.mark.parametrize("S,sizes,mapped", [(1, [40], False), (5, [300, 0, 77, 1], True), (128, [500, 3, 0, 9, 1, 2, 3, 90], True), (30, [2048], False), (3, [64, 128] * 5, False)])      # (at most 33 of M / 64 + experts)
def test_ffn_plan_of_small_calls(lib, S, sizes, mapped):
    """Calls with few groups and rows are planned by a kernel of their own: the same rows as with the general one, which the same groups take as
    soon as M, the bound of the rows, is larger."""
    say("ffn plan of small calls", S, sizes)
    d, f, E_loc = 256, 256, len(sizes)
    rng = np.random.default_rng(S + E_loc)
    parts = np.stack([rng.multinomial(n, np.full(S, 1.0 / S)) for n in sizes], axis=1)
    off = np.concatenate([[0], np.cumsum(parts.ravel())]).astype(np.int32)
    M, spare = int(off[-1]), 4096
    w = workloads.ffn_weights_on_device(E_loc, d, f, S, "bf16", DEV)
    x = workloads.activations_on_device(M + spare, d, S + 1, DEV)
    row_map = dev(np.concatenate([rng.permutation(M), np.arange(M, M + spare)]).astype(np.int32))
    gate = torch.rand((M + spare,), device=DEV)
    out = []
    lib.moe_ffn_tile_override(64)
    lib.moe_kernel_timing_enable(True)
    try:
        for rows, name in ((M, "ffn_small_plan_kernel"), (M + spare, "ffn_plan_kernel")):
            y = torch.zeros((rows, d), dtype=torch.bfloat16, device=DEV)
            if mapped:
                lib.moe_expert_ffn_sliced_mapped(x[:rows], dev(off), S, E_loc, row_map=row_map[:rows].contiguous(), row_gate=gate[:rows].contiguous(), y=y, **w)
            else:
                lib.moe_expert_ffn_sliced(x[:rows], dev(off), S, E_loc, y=y, **w)
            torch.cuda.synchronize()
            assert name in lib.moe_kernel_timing_read()
            out.append(y[:M])
    finally:
        lib.moe_kernel_timing_enable(False)
        lib.moe_ffn_tile_override()
    assert torch.equal(out[0], out[1]) and bool(out[0].abs().sum() > 0)


@pytest.mark.parametrize("dtype,tile_rows", [("bf16", 0), ("bf16", 64), ("bf16", 128), ("bf16", 256), ("fp8", 128)])
@pytest.mark.parametrize("S,E_loc", [(1, 3), (4, 1), (3, 2), (1, 1)])
def test_ffn_first_group_later(lib, dtype, tile_rows, S, E_loc):
    """A schedule whose first group begins behind row 0: its rows are the same as in a buffer that begins there, by every kernel and
    whether the rows are listed (several slices and experts) or not; the rows before it stay untouched."""
    say("ffn first group later", dtype, tile_rows, S, E_loc)
    d, f, skip, M = 256, 256, 37, 700
    w = workloads.ffn_weights_on_device(E_loc, d, f, S + E_loc, dtype, DEV)
    offsets = workloads.random_offsets(S * E_loc, M, seed=S + 7 * E_loc)
    x = workloads.activations_on_device(M + skip, d, 5, DEV)
    lib.moe_ffn_tile_override(tile_rows)
    try:
        y = lib.moe_expert_ffn_sliced(x, dev(offsets + skip), S, E_loc, y=torch.full_like(x, 3.0), **w)
        want = lib.moe_expert_ffn_sliced(x[skip:].clone(), dev(offsets), S, E_loc, **w)
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    assert torch.equal(y[skip:].view(torch.int16), want.view(torch.int16)) and bool((y[:skip] == 3.0).all())
    if dtype == "bf16" and tile_rows == 0:
        dy = workloads.activations_on_device(M + skip, d, 6, DEV)
        got = lib.moe_expert_ffn_backward_sliced(x, dy, dev(offsets + skip), S, E_loc, **w)
        want = lib.moe_expert_ffn_backward_sliced(x[skip:].clone(), dy[skip:].clone(), dev(offsets), S, E_loc, **w)
        torch.cuda.synchronize()
        assert torch.equal(got["dx"][skip:], want["dx"])
        for k in ("dw_gate", "dw_up", "dw_down"):
            assert torch.equal(got[k], want[k]), k


# ------------------------------------------------------------------------------ FFN backward
def check_backward(lib, E_loc, d, f, M, S, seed, what, spare=0, empty_frac=0.15):
    W = workloads.ffn_weights(E_loc, d, f, seed=seed)
    x = workloads.activations(M + spare, d, seed=seed + 1)
    dy = workloads.activations(M + spare, d, seed=seed + 2)
    offsets = workloads.random_offsets(S * E_loc, M, seed=seed + 3, empty_frac=empty_frac)
    w = upload_weights(W)
    out = lib.moe_expert_ffn_backward_sliced(dev_bf16(x), dev_bf16(dy), dev(offsets), S, E_loc, w["w_gate"], w["w_up"], w["w_down"])
    torch.cuda.synchronize()
    dx, dWg, dWu, dWd = oracle.expert_ffn_backward_sliced(x, dy, offsets, E_loc, W)
    if M > 0:
        check_ffn_error(ffn_error(host_bf16_bits(out["dx"])[:M], dx, offsets), "bf16", what + " dx")
    for name, ref in (("dw_gate", dWg), ("dw_up", dWu), ("dw_down", dWd)):
        got = oracle.decode_bf16(host_bf16_bits(out[name]))
        for e in range(E_loc):
            scale = np.abs(ref[e]).max()
            if scale == 0:
                assert not got[e].any(), (name, e)
                continue
            check_ffn_error(float(np.abs(got[e] - ref[e]).max() / scale), "bf16", "%s %s[%d]" % (what, name, e))
    return out


@pytest.mark.parametrize("E_loc,d,f,M,S", [(1, 256, 256, 300, 1), (2, 256, 384, 1500, 3), (4, 512, 640, 5000, 4), (3, 256, 1408, 900, 2)])
def test_ffn_backward_small(lib, E_loc, d, f, M, S):
    """dx for every row and the three weight gradients of every expert against the float64 chain rule."""
    say("ffn backward small", E_loc, d, f, M, S)
    check_backward(lib, E_loc, d, f, M, S, seed=d + f + M, what="small", spare=5)


@pytest.mark.parametrize("E_loc,d,f", [(40, 256, 256), (20, 256, 640), (12, 768, 384), (6, 1280, 256), (3, 2304, 1152), (2, 256, 4352)])
def test_ffn_backward_tickets(lib, E_loc, d, f):
    """Chunks of 2, 8 (5 used), 16 (9 used), 16 (10 used), 32 (30 used) and 32 places in the queues of the weight gradients, one and several chunks per
    product: every tile of every expert is computed."""
    say("ffn backward tickets", E_loc, d, f)
    check_backward(lib, E_loc, d, f, 700, 2, seed=d + f, what="tickets", empty_frac=0.3)


@pytest.mark.parametrize("S,M,E_loc", [(0, 0, 3), (0, 40, 3), (0, 40, 1100), (0, 40, 2100), (5, 0, 3)])
def test_ffn_backward_without_groups(lib, S, M, E_loc):
    """No slices (also with more experts than the planning workgroup has threads, or keeps in LDS) or no rows: zero weight gradients and
    nothing else is launched, since without groups there are no row boundaries to plan from."""
    say("ffn backward without groups", S, M, E_loc)
    d, f = 256, 256
    w = [torch.ones(sh, dtype=torch.bfloat16, device=DEV) for sh in ((E_loc, f, d), (E_loc, f, d), (E_loc, d, f))]
    x = torch.ones((M, d), dtype=torch.bfloat16, device=DEV)
    offsets = torch.zeros((S * E_loc + 1,), dtype=torch.int32, device=DEV)
    lib.moe_kernel_timing_enable(True)
    try:
        out = lib.moe_expert_ffn_backward_sliced(x, x.clone(), offsets, S, E_loc, *w)
        torch.cuda.synchronize()
        names = lib.moe_kernel_timing_read()
    finally:
        lib.moe_kernel_timing_enable(False)
    assert set(names) == {"bwd_zero_kernel"}
    assert not any(bool(out[k].any()) for k in ("dw_gate", "dw_up", "dw_down"))


@pytest.mark.parametrize("E_loc,M", [(1, 1023), (1, 1024), (1, 2100), (2, 4500), (1, 4200), (1, 9000), (1, 16500)])
def test_ffn_backward_parts(lib, E_loc, M):
    """Contractions of the weight gradients over a few hundred rows up to many parts of at least 768 rows: three slices' rows listed, remainders."""
    check_backward(lib, E_loc, 256, 256, M, 3, M, "parts")


@pytest.mark.parametrize("M", [1024, 1500, 2047])
def test_ffn_backward_sums_below_2048_rows_are_exact(lib, M):
    """The sums of an expert's rows, in one part or in two (from 1536 rows), are fp32: with the same x in every row and dy of +1 for the first half
    (and three more rows), -1 for the rest, dw_down is a small multiple of h, which a partial sum rounded to bf16 would lose
    (half the rows times h keeps 8 bits).  Every fp32 sum here is a multiple of h below 2^11 h: exact."""
    say("ffn backward exact sums", M)
    d, f = 256, 256
    w = upload_weights(workloads.ffn_weights(1, d, f, seed=M))
    x = dev_bf16(workloads.activations(1, d, seed=M)).expand(M, d).contiguous()
    dy = torch.full((M, d), -1.0, dtype=torch.bfloat16, device=DEV)
    dy[: M // 2 + 3] = 1.0
    run = lambda n: lib.moe_expert_ffn_backward_sliced(x[:n], dy[:n], dev(np.array([0, n], dtype=np.int32)), 1, 1, w["w_gate"], w["w_up"], w["w_down"])
    h = run(1)["dw_down"].float()                                          # one row, dy = 1: h itself
    got = run(M)["dw_down"]
    torch.cuda.synchronize()
    assert torch.equal(got, (h * (2 * (M // 2 + 3) - M)).to(torch.bfloat16))


def test_ffn_backward_rows_addressed_with_64_bits(lib):
    """x and dy above 4 GiB with several slices and experts: the rows of the plan are listed, and gathered (dh, dg, du, h) and scattered
    (dx) with 64-bit addresses.  Every row and gradient against float32 products of the GPU."""
    say("ffn backward, listed rows above 4 GiB")
    E_loc, d, f, S = 2, 8192, 256, 3
    M = (1 << 32) // (2 * d) + 1500
    offsets = workloads.random_offsets(S * E_loc, M, seed=51, empty_frac=0.0)
    w = {k: v for k, v in workloads.ffn_weights_on_device(E_loc, d, f, 52, "bf16", DEV).items()}
    x, dy = workloads.activations_on_device(M, d, 53, DEV), workloads.activations_on_device(M, d, 54, DEV)
    out = lib.moe_expert_ffn_backward_sliced(x, dy, dev(offsets), S, E_loc, **w)
    torch.cuda.synchronize()

    def check(got, ref, what):
        diff = (got.float() - ref).abs_()
        check_ffn_error(float(diff.max() / ref.abs().max()), "bf16", what)
        assert float(diff.norm() / ref.norm()) <= 1.2e-2, what               # (four roundings to bf16 of 2^-9 each, as elsewhere)

    for e in range(E_loc):
        wg, wu, wd = (w[k][e].float() for k in ("w_gate", "w_up", "w_down"))
        dWg, dWu, dWd = torch.zeros_like(wg), torch.zeros_like(wu), torch.zeros_like(wd)
        for s in range(S):
            lo, hi = int(offsets[s * E_loc + e]), int(offsets[s * E_loc + e + 1])
            xs, ds = x[lo:hi].float(), dy[lo:hi].float()
            g, u, dh = xs @ wg.t(), xs @ wu.t(), ds @ wd
            sig = torch.sigmoid(g)
            du, dg = dh * g * sig, dh * u * sig * (1 + g * (1 - sig))
            check(out["dx"][lo:hi], dg @ wg + du @ wu, "dx of slice %d, expert %d" % (s, e))
            dWg += dg.t() @ xs; dWu += du.t() @ xs; dWd += ds.t() @ (g * sig * u)
            del xs, ds
        for k, ref in (("dw_gate", dWg), ("dw_up", dWu), ("dw_down", dWd)):
            check(out[k][e], ref, "%s[%d]" % (k, e))


@pytest.mark.parametrize("f,S,sizes", [
    (256, 1, [64]), (384, 1, [129]),                                     # one expert: whole slabs, a remainder; rows in order
    (384, 2, [0, 1, 63, 64, 65, 127, 128, 192]),                         # slabs of 64 rows and their remainders, one slab, two, three; listed rows
    (256, 3, [1536, 200, 1600]), (640, 1, [1535, 5]), (256, 2, [40000])])    # the last experts split over parts with a remainder, or just not
def test_ffn_backward_weight_gradient_slabs(lib, f, S, sizes):
    """Ends of the contraction over an expert's rows, and rows that belong to other experts and hold infinities: they must not be touched, not
    even multiplied by zero."""
    say("ffn backward weight gradient slabs", f, S, sizes)
    d, E_loc = 256, len(sizes)
    W = workloads.ffn_weights(E_loc, d, f, seed=f + S)
    w = upload_weights(W)
    parts = np.array([[n // S + (s < n % S) for n in sizes] for s in range(S)])
    off = np.concatenate([[0], np.cumsum(parts.ravel())]).astype(np.int32)
    M = int(off[-1])
    x, dy = workloads.activations(M, d, seed=f + 1), workloads.activations(M, d, seed=f + 2)
    ref = oracle.expert_ffn_backward_sliced(x, dy, off, E_loc, W)[1:]
    bad = E_loc // 2 if E_loc > 1 else -1                             # this expert's rows
    xd, dyd = dev_bf16(x), dev_bf16(dy)
    for s in range(S):
        if bad >= 0:
            xd[off[s * E_loc + bad]:off[s * E_loc + bad + 1]] = float("inf")
            dyd[off[s * E_loc + bad]:off[s * E_loc + bad + 1]] = float("inf")
    out = lib.moe_expert_ffn_backward_sliced(xd, dyd, dev(off), S, E_loc, w["w_gate"], w["w_up"], w["w_down"])
    torch.cuda.synchronize()
    for name, want in zip(("dw_gate", "dw_up", "dw_down"), ref):
        got = oracle.decode_bf16(host_bf16_bits(out[name]))
        for e in range(E_loc):
            if e == bad:
                continue
            if sizes[e] == 0:
                assert not got[e].any(), (name, e)
            else:
                check_ffn_error(float(np.abs(got[e] - want[e]).max() / np.abs(want[e]).max()), "bf16", "%s[%d] of %s" % (name, e, sizes))


@pytest.mark.parametrize("d,f,sizes", [(1024, 512, [8000, 8000, 7999, 8001, 8000, 3]), (256, 256, test_parts.MANY[0])])
def test_ffn_backward_experts_without_room_for_sums(lib, d, f, sizes):
    """More parts are asked for than there are places for their sums: the last experts stay whole, those before them are split.  The second call is one
    whose experts ask for more parts than the table of them holds.  Against float32 products of the GPU."""
    say("ffn backward experts without room for sums", d, f, len(sizes), sum(sizes))
    E_loc, M = len(sizes), sum(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    w = workloads.ffn_weights_on_device(E_loc, d, f, d + f, "bf16", DEV)
    x, dy = workloads.activations_on_device(M, d, 81, DEV), workloads.activations_on_device(M, d, 82, DEV)
    out = lib.moe_expert_ffn_backward_sliced(x, dy, dev(off), 1, E_loc, **w)
    torch.cuda.synchronize()
    worst = 0.0
    for e in range(E_loc):
        wg, wu, wd = (w[k][e].float() for k in ("w_gate", "w_up", "w_down"))
        xs, ds = x[off[e]:off[e + 1]].float(), dy[off[e]:off[e + 1]].float()
        g, u, dh = xs @ wg.t(), xs @ wu.t(), ds @ wd
        sig = torch.sigmoid(g)
        for k, ref in (("dw_gate", (dh * u * sig * (1 + g * (1 - sig))).t() @ xs), ("dw_up", (dh * g * sig).t() @ xs), ("dw_down", ds.t() @ (g * sig * u))):
            diff = (out[k][e].float() - ref).abs()
            worst = max(worst, float(diff.max() / ref.abs().max()))
            assert float(diff.norm() / ref.norm()) <= 1.2e-2, (k, e)           # (four roundings to bf16 of 2^-9 each, as elsewhere)
    check_ffn_error(worst, "bf16", "all experts")


@pytest.mark.parametrize("tile_rows,kernels", [(64, 0), (128, 0), (256, 1), (256, 0)])
@pytest.mark.parametrize("d,f,S,sizes", [(256, 384, 3, [300, 0, 1, 64]), (512, 1664, 1, [65, 130]), (1536, 256, 2, [129, 7])])
def test_ffn_backward_row_products(lib, tile_rows, kernels, d, f, S, sizes):
    """dh, the gradient read-out and dx in tiles of every height (listed rows and rows in order, contractions split over workgroups where d or 2 f
    are long), twice with the same bits, against the float64 chain rule."""
    say("ffn backward row products", tile_rows, kernels, d, f, S, sizes)
    E_loc, M = len(sizes), sum(sizes)
    rng = np.random.default_rng(d + f)
    parts = np.stack([rng.multinomial(n, np.full(S, 1.0 / S)) for n in sizes], axis=1)
    off = np.concatenate([[0], np.cumsum(parts.ravel())]).astype(np.int32)
    W = workloads.ffn_weights(E_loc, d, f, seed=d + f)
    w = upload_weights(W)
    x, dy = workloads.activations(M, d, seed=f + 1), workloads.activations(M, d, seed=f + 2)
    lib.moe_ffn_tile_override(tile_rows, kernels)
    try:
        out, again = [lib.moe_expert_ffn_backward_sliced(dev_bf16(x), dev_bf16(dy), dev(off), S, E_loc, w["w_gate"], w["w_up"], w["w_down"]) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        lib.moe_ffn_tile_override()
    ref = oracle.expert_ffn_backward_sliced(x, dy, off, E_loc, W)
    check_ffn_error(ffn_error(host_bf16_bits(out["dx"]), ref[0], off), "bf16", "dx")
    for name, want in zip(("dw_gate", "dw_up", "dw_down"), ref[1:]):
        got = oracle.decode_bf16(host_bf16_bits(out[name]))
        for e in range(E_loc):
            if sizes[e]:
                check_ffn_error(float(np.abs(got[e] - want[e]).max() / np.abs(want[e]).max()), "bf16", "%s[%d]" % (name, e))
    assert all(torch.equal(out[k], again[k]) for k in out)


@pytest.mark.parametrize("tile_rows,kernels", [(0, 0), (64, 0), (128, 0), (256, 1)])
@pytest.mark.parametrize("d,f,S,sizes", [(256, 256, 1, [1536, 1]), (512, 1664, 2, [700, 90]), (256, 384, 3, [40000, 200]), (1024, 512, 1, [9000, 8000])])
def test_ffn_backward_stays_inside_its_workspace(lib, tile_rows, kernels, d, f, S, sizes):
    """A workspace of just the stated size, in front of bytes that are looked at afterwards: more of it changes no bit.  One without places for partial sums serves
    as well, with whole contractions; one without room for the tables and operands is refused."""
    say("ffn backward stays inside its workspace", tile_rows, d, f, S, sizes)
    E_loc, M = len(sizes), sum(sizes)
    rng = np.random.default_rng(d + f)
    parts = np.stack([rng.multinomial(n, np.full(S, 1.0 / S)) for n in sizes], axis=1)
    off = dev(np.concatenate([[0], np.cumsum(parts.ravel())]).astype(np.int32))
    w = workloads.ffn_weights_on_device(E_loc, d, f, d + f, "bf16", DEV)
    x, dy = workloads.activations_on_device(M, d, 91, DEV), workloads.activations_on_device(M, d, 92, DEV)
    need = int(lib.load().moe_ffn_backward_workspace_bytes(M, E_loc, d, f))
    room = torch.full((need + (64 << 20),), 0xA5, dtype=torch.uint8, device=DEV)
    lib.moe_ffn_tile_override(tile_rows, kernels)
    try:
        just = lib.moe_expert_ffn_backward_sliced(x, dy, off, S, E_loc, **w, workspace=room[:need])
        torch.cuda.synchronize()
        assert bool((room[need:] == 0xA5).all())
        more = lib.moe_expert_ffn_backward_sliced(x, dy, off, S, E_loc, **w, workspace=room)
        torch.cuda.synchronize()
        tiles = f // 128 * (d // 256) + d // 256 * -(-f // 256)
        places = min(1024, M // 768 * tiles)
        least = need - max((places << 18) if places >= 2 * tiles else 0, (32 << 20) if max(d, 2 * f) >= 1536 else 0)
        room.fill_(0xA5)
        whole = lib.moe_expert_ffn_backward_sliced(x, dy, off, S, E_loc, **w, workspace=room[:least])
        torch.cuda.synchronize()
        assert bool((room[least:] == 0xA5).all())
        with pytest.raises(lib.MoeError):
            lib.moe_expert_ffn_backward_sliced(x, dy, off, S, E_loc, **w, workspace=room[:least - 1])
    finally:
        lib.moe_ffn_tile_override()
    assert all(float((just[k].float() - whole[k].float()).norm() / whole[k].float().norm()) <= 2.0 ** -7 for k in just)      # (dh, dg and du round to bf16 in between)
    assert all(torch.equal(just[k], more[k]) for k in just)


def test_ffn_backward_edge_cases(lib):
    say("ffn backward edge cases")
    # an expert without rows (zero weight gradients), a single row, no rows at all
    E_loc, d, f = 3, 256, 256
    W = workloads.ffn_weights(E_loc, d, f, seed=3)
    w = upload_weights(W)
    x = workloads.activations(40, d, seed=4)
    dy = workloads.activations(40, d, seed=5)
    for sizes in ([40, 0, 0], [0, 1, 0], [0, 0, 0], [13, 0, 27]):
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        out = lib.moe_expert_ffn_backward_sliced(dev_bf16(x), dev_bf16(dy), dev(off), 1, E_loc, w["w_gate"], w["w_up"], w["w_down"])
        torch.cuda.synchronize()
        dx, dWg, dWu, dWd = oracle.expert_ffn_backward_sliced(x, dy, off, E_loc, W)
        n = int(off[-1])
        if n:
            check_ffn_error(ffn_error(host_bf16_bits(out["dx"])[:n], dx, off), "bf16", str(sizes))
        for name, ref in (("dw_gate", dWg), ("dw_up", dWu), ("dw_down", dWd)):
            got = oracle.decode_bf16(host_bf16_bits(out[name]))
            for e in range(E_loc):
                if sizes[e] == 0:
                    assert not got[e].any(), (sizes, name, e)
                else:
                    assert np.abs(got[e] - ref[e]).max() <= FFN_GUARD["bf16"] * np.abs(ref[e]).max(), (sizes, name, e)
    with pytest.raises(lib.MoeError):                                    # f below the smallest supported width
        lib.moe_expert_ffn_backward_sliced(dev_bf16(x), dev_bf16(dy), dev(off), 1, E_loc, w["w_gate"][:, :128].contiguous(),
                                           w["w_up"][:, :128].contiguous(), w["w_down"][:, :, :128].contiguous())


def test_ffn_backward_many_tiles(lib):
    """A schedule on which every workgroup runs several tiles in each of the six matrix launches."""
    say("ffn backward many tiles")
    check_backward(lib, 4, 1536, 768, 36000, 6, seed=61, what="36000 rows")


def test_whole_path_backward_c2(lib):
    """c2's hottest receiving rank: the schedule from the GPU path, then the backward pass of its FFN; every row of dx and
    all twelve weight gradients against the oracle."""
    say("whole path backward c2")
    cfg = workloads.CONFIGS["c2"]
    ids = workloads.config_routing(cfg)
    d_ids = dev(ids)
    traffic, _ = lib.moe_route_histogram(d_ids, cfg.E)
    r = int(traffic.sum(0).argmax().item())
    sched = lib.moe_decompose_greedy(traffic.unsqueeze(0), cfg.kmax, zero_diag=True)
    offsets = lib.moe_slice_table(d_ids, cfg.E, r, traffic, sched["perms"][0], sched["durations"][0], sched["counts"], cfg.kmax)
    torch.cuda.synchronize()
    off = offsets.cpu().numpy()
    M = int(off[-1])
    W, Wd = config_weights(cfg)
    x = workloads.activations(M, cfg.d, seed=cfg.seed + 3)
    dy = workloads.activations(M, cfg.d, seed=cfg.seed + 4)
    out = lib.moe_expert_ffn_backward_sliced(dev_bf16(x), dev_bf16(dy), offsets, cfg.kmax + 2, cfg.E_loc, Wd["w_gate"], Wd["w_up"], Wd["w_down"])
    torch.cuda.synchronize()
    dx, dWg, dWu, dWd = oracle.expert_ffn_backward_sliced(x, dy, off, cfg.E_loc, W)
    check_ffn_error(ffn_error(host_bf16_bits(out["dx"]), dx, off), "bf16", "dx, all %d rows" % M)
    for name, ref in (("dw_gate", dWg), ("dw_up", dWu), ("dw_down", dWd)):
        got = oracle.decode_bf16(host_bf16_bits(out[name]))
        for e in range(cfg.E_loc):
            check_ffn_error(float(np.abs(got[e] - ref[e]).max() / np.abs(ref[e]).max()), "bf16", "%s[%d]" % (name, e))
    _WEIGHTS.clear()


# ------------------------------------------------------------------------------ combine
def combine_tolerance(y_bits, row_of, gate, ref):
    """fp32 accumulation of topk terms (2^-24 of the terms' magnitudes each) and one rounding to bf16 (2^-9 of the
    result): |out - ref| <= 2^-8 |ref| + 2^-20 sum_j |gate * y| elementwise, with room to spare."""
    y = np.abs(oracle.decode_bf16(y_bits))
    live = (row_of >= 0) & (row_of < y.shape[0])
    g = np.ones(row_of.shape, dtype=np.float64) if gate is None else np.abs(gate.astype(np.float64))
    mag = (y[np.clip(row_of, 0, y.shape[0] - 1)] * (g * live)[:, :, None]).sum(axis=1)
    return 2.0 ** -8 * np.abs(ref) + 2.0 ** -20 * mag + 1e-30


@pytest.mark.parametrize("T,topk,d,R", [(1, 1, 8, 1), (37, 2, 256, 80), (50, 3, 2056, 160), (19, 8, 4096, 200), (300, 4, 7168, 1200),
                                       (11, 6, 512, 70), (5, 5, 16, 40)])
@pytest.mark.parametrize("gated", [True, False])
def test_combine_topk_sum(lib, T, topk, d, R, gated):
    say("combine", T, topk, d, R, gated)
    rng = np.random.default_rng(T * 31 + topk)
    y = workloads.activations(R, d, seed=T + d)
    row_of = rng.integers(0, R, size=(T, topk)).astype(np.int32)
    if T > 4:
        row_of[1, 0] = -1                                              # a dropped assignment
        row_of[2, :] = -1                                              # a token that lost every expert
        row_of[3, topk - 1] = R + 5                                    # past the end: ignored as well
    gate = rng.uniform(0.0, 1.0, size=(T, topk)).astype(np.float32) if gated else None
    out0 = torch.full((T, d), 3.0, dtype=torch.bfloat16, device=DEV)
    out = lib.moe_combine_topk_sum(dev_bf16(y), dev(row_of), dev(gate) if gated else None, out=out0)
    torch.cuda.synchronize()
    ref = oracle.combine_topk_sum(y, row_of, gate)
    got = oracle.decode_bf16(host_bf16_bits(out))
    assert (np.abs(got - ref) <= combine_tolerance(y, row_of, gate, ref)).all(), np.abs(got - ref).max()
    if T > 4:
        assert not got[2].any()


def test_moe_layer_dispatch_compute_combine(lib):
    """One whole layer on one GPU (every expert local): tokens -> one row per (token, expert) assignment -> slice table
    with row map -> FFN with fused gather, scatter and router weight -> weighted top-k sum per token; against
    sum_j gate[t][j] * FFN_{e(t,j)}(x_t) evaluated by the oracle."""
    say("moe layer: dispatch -> compute -> combine")
    T, E, topk, d, f = 3000, 4, 2, 512, 384
    ids = workloads.route_topk(1, T, E, topk, 1.0, seed=77)
    rng = np.random.default_rng(78)
    gate = rng.uniform(0.1, 1.0, size=(T, topk)).astype(np.float32)
    W = workloads.ffn_weights(E, d, f, seed=79)
    x_tok = workloads.activations(T, d, seed=80)
    x_arr = np.repeat(x_tok, topk, axis=0)                               # arrival order: (token, slot)
    d_ids = dev(ids)
    traffic, _ = lib.moe_route_histogram(d_ids, E)
    kmax = 2
    sched = lib.moe_decompose_greedy(traffic.unsqueeze(0), kmax, zero_diag=True)
    M = T * topk
    offsets, arr, asg = lib.moe_slice_table_rows(d_ids, E, 0, traffic, sched["perms"][0], sched["durations"][0], sched["counts"], kmax, M)
    torch.cuda.synchronize()
    assert int(offsets[-1].item()) == M and torch.equal(arr, asg)        # one source: arrival index = assignment index
    row_gate = dev(gate.reshape(-1))[arr.long()].contiguous()            # router weight of the assignment behind each schedule row
    y_arr = lib.moe_expert_ffn_sliced_mapped(dev_bf16(x_arr), offsets, kmax + 2, E, row_map=arr, row_gate=row_gate, **upload_weights(W))
    row_of = np.arange(M, dtype=np.int32).reshape(T, topk)
    out = lib.moe_combine_topk_sum(y_arr, dev(row_of))
    torch.cuda.synchronize()
    # oracle: every assignment through its expert, then the weighted sum
    off_e = np.zeros(E + 1, dtype=np.int32)
    flat = ids.reshape(-1)
    order = np.argsort(flat, kind="stable")
    off_e[1:] = np.cumsum(np.bincount(flat, minlength=E))
    y_sorted = oracle.expert_ffn_sliced(x_arr[order], off_e, E, W)
    y_asg = np.empty_like(y_sorted)
    y_asg[order] = y_sorted
    ref = (y_asg.reshape(T, topk, d) * gate.astype(np.float64)[:, :, None]).sum(axis=1)
    got = oracle.decode_bf16(host_bf16_bits(out))
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    check_ffn_error(err, "bf16", "layer output, %d tokens" % T)


def sample_rows(off, per_group, seed=1, blocks=()):
    """Every non-empty group contributes its first and last rows plus a random sample; `blocks` adds every row of the
    given (first row, end row) stretches."""
    rng = np.random.default_rng(seed)
    off = np.asarray(off, dtype=np.int64)
    rows = []
    for g in range(len(off) - 1):
        lo, hi = off[g], off[g + 1]
        if hi > lo:
            rows += [lo, hi - 1] + list(rng.integers(lo, hi, size=min(per_group, hi - lo)))
    for lo, hi in blocks:
        rows += list(range(int(lo), int(hi)))
    return np.unique(np.array(rows, dtype=np.int64))


def whole_tiles(off, want, tile=256):
    """Row stretches covering whole 256-row tiles: the first tile of every large group, a tile from the middle of the
    largest group, and the ragged last tiles of the groups -- `want` stretches in all (fewer if the schedule is small)."""
    off = np.asarray(off, dtype=np.int64)
    size = np.diff(off)
    firsts = [(off[g], min(off[g] + tile, off[g + 1])) for g in np.argsort(-size, kind="stable") if size[g] >= tile]
    tails = [(off[g] + (size[g] - 1) // tile * tile, off[g + 1]) for g in np.argsort(-size, kind="stable") if size[g] > tile and size[g] % tile]
    g = int(np.argmax(size))
    mid = [(off[g] + size[g] // tile // 2 * tile, min(off[g] + (size[g] // tile // 2 + 1) * tile, off[g + 1]))] if size[g] >= 3 * tile else []
    out, k = [], 0
    while len(out) < want and (k < len(firsts) or k < len(tails) or k < len(mid)):
        for lst in (firsts, tails, mid):
            if k < len(lst) and len(out) < want:
                out.append(lst[k])
        k += 1
    return out


def test_whole_path_with_row_map_c2(lib):
    """c2 at full size: rows arrive source by source; slice table -> row map -> FFN with fused gather / scatter.
    Every row is compared."""
    say("whole path with row map, c2")
    cfg = workloads.CONFIGS["c2"]
    ids = workloads.config_routing(cfg)
    d_ids = dev(ids)
    traffic, _ = lib.moe_route_histogram(d_ids, cfg.E)
    r = int(traffic.sum(0).argmax().item())
    sched = lib.moe_decompose_greedy(traffic.unsqueeze(0), cfg.kmax, zero_diag=True)
    M = int(traffic[:, r].sum().item())
    offsets, arr, asg = lib.moe_slice_table_rows(d_ids, cfg.E, r, traffic, sched["perms"][0], sched["durations"][0],
                                                 sched["counts"], cfg.kmax, M)
    W = workloads.ffn_weights(cfg.E_loc, cfg.d, cfg.f, seed=cfg.seed, dtype=cfg.weight_dtype)
    x = workloads.activations(M, cfg.d, seed=cfg.seed + 1)                                # arrival order
    gate = np.random.default_rng(5).uniform(0.05, 1.0, size=M).astype(np.float32)
    y = lib.moe_expert_ffn_sliced_mapped(dev_bf16(x), offsets, cfg.kmax + 2, cfg.E_loc, row_map=arr, row_gate=dev(gate),
                                         **upload_weights(W))
    torch.cuda.synchronize()
    th = traffic.cpu().numpy()
    rp, rd, _ = oracle.decompose_greedy(th, cfg.kmax, zero_diag=True)
    ref_off, ref_rows = oracle.slice_table(ids, cfg.E, r, th, rp, rd, cfg.kmax)
    assert np.array_equal(offsets.cpu().numpy(), ref_off) and np.array_equal(asg.cpu().numpy(), ref_rows)
    row_map = np.searchsorted(np.sort(ref_rows), ref_rows)
    ref, target = oracle.expert_ffn_sliced_mapped(x, ref_off, cfg.E_loc, W, row_map, gate)
    assert np.array_equal(np.sort(target), np.arange(M))
    check_ffn_error(ffn_error(host_bf16_bits(y)[target], ref, ref_off), "bf16", "all %d rows" % M)


# ------------------------------------------------------------------------------ whole path, full-size configs
_WEIGHTS = {}


def config_weights(cfg):
    """(host weights, uploaded weights) of a named config, drawn once per test session (the fp8 set takes half a minute)."""
    if cfg.name not in _WEIGHTS:
        W = workloads.ffn_weights(cfg.E_loc, cfg.d, cfg.f, seed=cfg.seed, dtype=cfg.weight_dtype)
        _WEIGHTS.clear()                                              # one set at a time on the device
        _WEIGHTS[cfg.name] = (W, upload_weights(W))
    return _WEIGHTS[cfg.name]


def test_whole_path_under_graph_capture(lib):
    """The library allocates nothing, copies nothing and clears nothing with runtime calls, so histogram -> greedy ->
    slice table (on the built-in work area) -> FFN can be recorded into a HIP graph once, with the row capacity as M
    (rows past offsets[last] are left alone), and replayed on new routings and activations.  Every replay is compared
    bit for bit with the same calls made eagerly on the same inputs (eager work and synchronisation between replays)."""
    say("whole path under graph capture")
    cfg = workloads.CONFIGS["tiny"]
    N, E, kmax, r = cfg.N, cfg.E, cfg.kmax, 3
    cap = N * cfg.T * cfg.topk                                         # no routing sends more rows than this to one rank
    W, Wd = config_weights(cfg)
    ids_s = torch.zeros((N, cfg.T, cfg.topk), dtype=torch.int32, device=DEV)
    x_s = torch.zeros((cap, cfg.d), dtype=torch.bfloat16, device=DEV)
    y_s = torch.zeros((cap, cfg.d), dtype=torch.bfloat16, device=DEV)
    traffic = torch.zeros((N, N), dtype=torch.int32, device=DEV)
    counts_e = torch.zeros((N, E), dtype=torch.int32, device=DEV)
    sched = dict(perms=torch.zeros((1, kmax, N), dtype=torch.uint8, device=DEV), durations=torch.zeros((1, kmax), dtype=torch.int32, device=DEV),
                 counts=torch.zeros((1,), dtype=torch.int32, device=DEV), residual=torch.zeros((1, N, N), dtype=torch.int32, device=DEV), hashes=None)
    offsets = torch.zeros(((kmax + 2) * cfg.E_loc + 1,), dtype=torch.int32, device=DEV)
    ws = torch.empty((lib.moe_ffn_workspace_bytes(cap, cfg.d, cfg.f),), dtype=torch.uint8, device=DEV)

    def path():
        lib.moe_route_histogram(ids_s, E, traffic=traffic, expert_counts=counts_e)
        lib.moe_decompose_greedy(traffic.view(1, N, N), kmax, zero_diag=True, out=sched)
        lib.moe_slice_table_static(ids_s, E, r, traffic, sched["perms"][0], sched["durations"][0], sched["counts"], kmax, offsets)
        lib.moe_expert_ffn_sliced(x_s, offsets, kmax + 2, cfg.E_loc, y=y_s, workspace=ws, **Wd)

    def load_inputs(seed):
        rng = np.random.default_rng(seed)
        ids_s.copy_(torch.from_numpy(rng.integers(0, E, size=(N, cfg.T, cfg.topk), dtype=np.int32)))
        x_s.copy_(workloads.activations_on_device(cap, cfg.d, 100 + seed, DEV))

    def clear():
        for t in (traffic, sched["perms"], sched["durations"], sched["counts"], sched["residual"], offsets):
            t.zero_()
        y_s.fill_(0.5)

    outputs = lambda: [t.clone() for t in (traffic, sched["perms"], sched["durations"], sched["counts"], sched["residual"], offsets, y_s)]
    load_inputs(0)
    path()                                                             # warm-up outside the capture (per-device kernel attributes)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        path()
    for seed in (1, 2, 3):
        load_inputs(seed)
        clear()
        path()
        torch.cuda.synchronize()
        eager = outputs()
        clear()                                                         # (entries past counts / offsets[last] are left alone by the calls)
        graph.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("traffic", "perms", "durations", "counts", "residual", "offsets", "y"), eager, outputs()):
            assert torch.equal(a, b), (seed, name)
        M = int(offsets[-1].item())
        assert 0 < M < cap and bool((y_s[M:] == 0.5).all())                 # rows past the schedule are untouched
    # one replay against the oracle as well (the eager path is what the other tests compare with it)
    off = offsets.cpu().numpy().astype(np.int64)
    rows = np.arange(int(off[-1]), dtype=np.int64)
    ref = oracle.expert_ffn_sliced(host_bf16_bits(x_s[: int(off[-1])]), off, cfg.E_loc, W, rows=rows)
    check_ffn_error(ffn_error(host_bf16_bits(y_s[: int(off[-1])]), ref, off, rows=rows), cfg.weight_dtype, "graph replay")


def run_path(lib, cfg, r, which="greedy", x_seed=0, x_on_device=False):
    """histogram -> decomposition -> slice table -> FFN on the GPU; returns everything on the host (x and y stay on
    the device when x_on_device: the checker reads back the rows it compares)."""
    ids = workloads.config_routing(cfg)
    d_ids = dev(ids)
    traffic, _ = lib.moe_route_histogram(d_ids, cfg.E)
    kmax = cfg.kmax if which == "greedy" else oracle.bvn_bound(cfg.N)
    fn = lib.moe_decompose_greedy if which == "greedy" else lib.moe_decompose_bvn
    sched = fn(traffic.unsqueeze(0), kmax, zero_diag=True)
    offsets = lib.moe_slice_table(d_ids, cfg.E, r, traffic, sched["perms"][0], sched["durations"][0], sched["counts"], kmax)
    torch.cuda.synchronize()
    M = int(offsets[-1].item())
    W, Wd = config_weights(cfg)
    if x_on_device:
        x = workloads.activations_on_device(M, cfg.d, cfg.seed + x_seed, DEV)
        xd = x
    else:
        x = workloads.activations(M, cfg.d, seed=cfg.seed + x_seed)
        xd = dev_bf16(x)
    say("   rows", M, "FFN call")
    y = lib.moe_expert_ffn_sliced(xd, offsets, kmax + 2, cfg.E_loc, **Wd)
    torch.cuda.synchronize()
    return dict(ids=ids, traffic=traffic.cpu().numpy(), sched={k: (v.cpu().numpy() if v is not None else None) for k, v in sched.items()},
                offsets=offsets.cpu().numpy(), M=M, W=W, x=x, y=y if x_on_device else host_bf16_bits(y), kmax=kmax)


def check_path(cfg, r, res, which, per_group=None, tiles=0):
    """Integer stages bit-exact; FFN on every row (per_group None) or on a sample: per_group random rows of every group,
    its first and last row, and every row of `tiles` whole 256-row tiles."""
    traffic, _ = oracle.route_histogram(res["ids"], cfg.E)
    assert np.array_equal(res["traffic"], traffic)
    kmax = res["kmax"]
    if which == "greedy":
        rp, rd, rr = oracle.decompose_greedy(traffic, kmax, zero_diag=True)
    else:
        rp, rd, rr, _, _ = oracle.decompose_bvn(traffic, kmax, zero_diag=True)
    c = int(res["sched"]["counts"][0])
    assert c == len(rd)
    assert np.array_equal(res["sched"]["perms"][0, :c], rp) and np.array_equal(res["sched"]["durations"][0, :c], rd)
    assert np.array_equal(res["sched"]["residual"][0], rr)
    ref_off, _ = oracle.slice_table(res["ids"], cfg.E, r, traffic, rp, rd, kmax, want_rows=False)
    assert np.array_equal(res["offsets"], ref_off)
    assert res["M"] == traffic[:, r].sum()
    off = res["offsets"].astype(np.int64)
    if per_group is None:
        rows = np.arange(res["M"], dtype=np.int64)
    else:
        rows = sample_rows(off, per_group, blocks=whole_tiles(off, tiles))
    if torch.is_tensor(res["x"]):                                     # x, y on the device: fetch the compared rows only
        idx = torch.from_numpy(rows).to(DEV)
        x_rows, y_rows = host_bf16_bits(res["x"][idx]), host_bf16_bits(res["y"][idx])
        ref = oracle.expert_ffn_sliced(_RowsView(x_rows, rows, res["M"]), off, cfg.E_loc, res["W"], rows=rows)
    else:
        y_rows = res["y"][rows]
        ref = oracle.expert_ffn_sliced(res["x"], off, cfg.E_loc, res["W"], rows=rows)
    check_ffn_error(ffn_error(y_rows, ref, off, rows=rows), cfg.weight_dtype, "%d of %d rows" % (len(rows), res["M"]))


class _RowsView:
    """Stands in for x[M][d] when only some rows are on the host: indexing with a subset of `rows` returns them."""
    def __init__(self, data, rows, M):
        self.data, self.rows, self.shape = data, rows, (M, data.shape[1])

    def __getitem__(self, idx):
        pos = np.searchsorted(self.rows, idx)
        assert np.array_equal(self.rows[pos], idx)
        return self.data[pos]


@pytest.mark.parametrize("name,which", [("tiny", "greedy"), ("tiny", "bvn"), ("c2", "greedy"), ("c2", "bvn")])
def test_whole_path_full_size(lib, name, which):
    """Hottest receiving rank (the rank the bench runs), every row compared."""
    cfg = workloads.CONFIGS[name]
    say("whole path", name, which)
    ids = workloads.config_routing(cfg)
    traffic, _ = oracle.route_histogram(ids, cfg.E)
    r = int(np.argmax(traffic.sum(0)))
    res = run_path(lib, cfg, r, which)
    check_path(cfg, r, res, which)


def test_whole_path_c3_hottest_rank(lib):
    """The 14336-wide expert on its hottest receiving rank (72 408 rows, the bench workload): at least 256 rows of every
    group and every row of 10 whole tiles."""
    cfg = workloads.CONFIGS["c3"]
    say("whole path c3, hottest rank")
    ids = workloads.config_routing(cfg)
    traffic, _ = oracle.route_histogram(ids, cfg.E)
    r = int(np.argmax(traffic.sum(0)))
    res = run_path(lib, cfg, r, "greedy")
    assert res["M"] == traffic[:, r].sum() and res["M"] > 70000
    check_path(cfg, r, res, "greedy", per_group=256, tiles=10)


@pytest.mark.parametrize("rank", ["median", "hottest"])
def test_whole_path_c4_fp8(lib, rank):
    """64 ranks, 256 experts, top-8, heavy skew, fp8 block-scaled weights.  The hottest receiving rank gets 529 867 rows
    (7.6 GB of activations: M * d > 2^31, drawn on the device); rows of every (slice, expert) group are compared."""
    cfg = workloads.CONFIGS["c4"]
    say("whole path c4 fp8,", rank, "rank")
    ids = workloads.config_routing(cfg)
    traffic, _ = oracle.route_histogram(ids, cfg.E)
    order = np.argsort(-traffic.sum(0), kind="stable")
    r = int(order[0]) if rank == "hottest" else int(order[len(order) // 2])
    res = run_path(lib, cfg, r, "greedy", x_on_device=(rank == "hottest"))
    if rank == "hottest":
        assert res["M"] * cfg.d > (1 << 31)
        check_path(cfg, r, res, "greedy", per_group=40, tiles=4)
    else:
        check_path(cfg, r, res, "greedy", per_group=16, tiles=2)
    _WEIGHTS.clear()


def test_decompose_stress_batch_hashes(lib):
    """A larger slice of the batched stress workload in count/hash-only mode: every schedule hash equals the
    oracle's, and the full batch size runs with sane counts."""
    say("decompose stress batch hashes")
    mats = workloads.stress_matrices(1024, 128)
    # (a batch this large takes the 16-bit residual by itself; two matrices get entries that do not fit and are redone)
    mats[5, 3, 77] = 70000
    mats[700] = mats[700] * 2
    assert mats[700].max() >= 65536
    out = lib.moe_decompose_greedy(dev(mats), 32, zero_diag=True, want_perms=False, want_residual=False, want_hashes=True)
    torch.cuda.synchronize()
    ref = oracle.decompose_batch("greedy", mats, 32, zero_diag=True, nthreads=16, want_perms=False, want_residual=False)
    assert np.array_equal(out["counts"].cpu().numpy(), ref["counts"])
    assert np.array_equal(out["hashes"].cpu().numpy().view(np.uint64), ref["hashes"])
    assert np.array_equal(out["durations"].cpu().numpy(), ref["durations"])
    big = torch.from_numpy(np.tile(mats, (8, 1, 1))).to(DEV)                 # 8192 matrices, the stress batch size
    out8 = lib.moe_decompose_greedy(big, 32, zero_diag=True, want_perms=False, want_residual=False, want_hashes=True)
    torch.cuda.synchronize()
    assert np.array_equal(out8["hashes"].cpu().numpy().view(np.uint64), np.tile(ref["hashes"], 8))

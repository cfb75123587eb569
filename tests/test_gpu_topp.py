"""Top-p (nucleus) features: exact cutoff index, rank and renormalised
features, HIP path vs the fp64 oracle."""

import ctypes as C
import math

import numpy as np
import pytest
import torch

import paper_2608_28726_amd as pr
from paper_2608_28726_amd import workloads as wl
from oracle import sequence as oseq
from tests.gpu_common import compare_features, gpu_features, oracle_features, require_gpu, to_dev
from tests.helpers import assert_floats

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _run(z, ids, T, P, dtype=torch.float32):
    logits, ids, T, P = to_dev(torch.as_tensor(z, dtype=torch.float32).to(dtype), torch.as_tensor(ids, dtype=torch.int32),
                               torch.as_tensor(T, dtype=torch.float32), torch.as_tensor(P, dtype=torch.float32))
    return logits, ids, T, P


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [2, 7, 8, 64, 1000, 32000])
def test_topp_random_rows(V, dtype):
    rng = np.random.default_rng(100 + V)
    n = 24
    z = rng.normal(0, rng.uniform(0.5, 4, (n, 1)), (n, V))
    z[np.arange(n), rng.integers(0, V, n)] += rng.uniform(0, 15, n)
    T = rng.uniform(0.3, 1.2, n)
    P = rng.uniform(0.05, 0.99, n)
    P[:4] = [1.0, 2.0, 1e-7, 0.999]
    ids = rng.integers(0, V, n)
    logits, ids, T, P = _run(z, ids, T, P, dtype)
    print(f"case topp random V={V} {dtype}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


def test_topp_special_rows():
    V = 64
    rows, ids, Ts, Ps = [], [], [], []
    def add(z, y, T, P):
        rows.append(np.asarray(z, dtype=np.float64)); ids.append(y); Ts.append(T); Ps.append(P)
    add(np.zeros(V), 3, 1.0, 0.5)            # uniform: k = 32
    add(np.zeros(V), 40, 1.0, 0.5)           # sampled token outside the nucleus
    add(np.zeros(V), 0, 1.0, 0.3)            # k = ceil(0.3 * 64) = 20
    z = np.full(V, -np.inf); z[5] = 1.0
    add(z, 5, 1.0, 0.9)                      # one-hot via -inf
    add(z, 6, 1.0, 0.9)                      # masked sampled token
    add(np.arange(V) * -0.5, 2, 0.7, 0.8)    # geometric
    add(np.zeros(V), 1, 1.0, 0.0)            # P = 0: flagged
    add(np.zeros(V), 1, 1.0, math.nan)       # P = NaN: flagged
    add(np.zeros(V), 1, 1.0, -0.5)           # P < 0: flagged
    add(np.where(np.arange(V) < 10, 2.0, 0.0), 9, 1.0, 0.5)   # tie block at the top
    logits, ids, T, P = _run(np.stack(rows), ids, Ts, Ps)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_undefined_rows_with_a_nucleus(dtype):
    """Rows with 0 < P < 1 whose distribution is undefined: their first pass
    forms no exps, so a NaN must still mark the row (in the vector body and
    in the scalar tail, V = 67); +inf and all -inf rows; a rejected
    temperature (the plain pass); one ordinary row as a control."""
    V = 67
    rng = np.random.default_rng(67)
    base = rng.normal(0, 1, (6, V))
    base[0, 10] = np.nan                     # NaN among the vectors
    base[1, 66] = np.nan                     # NaN in the tail
    base[2, 5] = np.inf                      # +inf
    base[3] = -np.inf                        # every token masked
    T = [1.0, 1.0, 1.0, 1.0, 0.0, 0.8]       # row 4: rejected temperature
    P = [0.9, 0.9, 0.9, 0.9, 0.9, 0.9]
    ids = [3, 4, 5, 6, 7, 8]
    logits, ids, T, P = _run(base, ids, T, P, dtype)
    print(f"case topp undefined rows {dtype}", flush=True)
    g = gpu_features(logits, ids, T, P)
    assert (g["flags"][:4] & pr.FLAG_NONFINITE).all() and g["flags"][4] & pr.FLAG_BAD_TP
    assert g["flags"][5] & (pr.FLAG_NONFINITE | pr.FLAG_BAD_TP) == 0
    compare_features(g, oracle_features(logits, ids, T, P))


@pytest.mark.parametrize("V", [262144, 151936])
def test_topp_massive_ties_radix_path(V):
    """Rows whose boundary bins hold more logits than the LDS sort takes:
    all-equal bf16 rows and rows with a few distinct values."""
    rng = np.random.default_rng(V)
    rows = [np.zeros(V), rng.choice([0.0, 0.5, 1.0], size=V), np.full(V, 3.0)]
    rows[2][: V // 3] = 3.5
    ids = [7, int(rng.integers(0, V)), V - 1]
    logits, ids, T, P = _run(np.stack(rows), ids, [1.0, 0.9, 1.1], [0.37, 0.8, 0.6], torch.bfloat16)
    print(f"case topp ties V={V}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


def test_topp_deterministic():
    """Two runs give bit-identical outputs on every path: the two-read
    method (random rows), the three-pass fallback (near-flat row) and its
    radix refinement (tie-heavy rows), whose float atomics only choose bins
    and digits."""
    V = 151936
    rng = np.random.default_rng(5)
    rows = [rng.normal(0, 2, V), rng.normal(0, 0.01, V), np.zeros(V), rng.choice([0.0, 0.5, 1.0], size=V)]
    ids = [int(rng.integers(0, V)) for _ in rows]
    logits, ids, T, P = _run(np.stack(rows), ids, [0.8, 1.2, 1.0, 0.9], [0.9, 0.93, 0.37, 0.8], torch.bfloat16)
    print("case topp deterministic", flush=True)
    a1 = gpu_features(logits, ids, T, P)
    a2 = gpu_features(logits, ids, T, P)
    for k in a1:
        assert np.array_equal(a1[k].view(np.uint32), a2[k].view(np.uint32)), k
    compare_features(a1, oracle_features(logits, ids, T, P))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_histogram_edge_rows(dtype):
    """Rows aimed at each branch of the two-read method: no finite anchor
    (the first vectors all -inf), more logits far above the anchor than the
    list holds, a crossing inside that list (one dominant spike), a nucleus
    spanning the list and the bins, a near-flat row with a wide window, and
    large logits on both sides of the limit on |A0| / T of the binning."""
    V = 65536
    rng = np.random.default_rng(77)
    rows, ids, Ts, Ps = [], [], [], []
    def add(z, y, T, P):
        rows.append(np.asarray(z, dtype=np.float64)); ids.append(int(y)); Ts.append(T); Ps.append(P)
    z = rng.normal(0, 2, V); z[:20000] = -np.inf
    add(z, 30000, 1.0, 0.9)                                  # no finite anchor among the first vectors
    z = rng.normal(0, 1, V); z[40000:41000] = 40.0 + rng.normal(0, 1, 1000)
    add(z, 40500, 1.0, 0.9)                                  # 1,000 logits ~40 nats above the anchor
    z = rng.normal(0, 1, V); z[50000] = 120.0
    add(z, 50000, 1.0, 0.9)                                  # one spike: nucleus = {spike}
    z = rng.normal(0, 1, V); z[60000] = 42.0
    add(z, 123, 4.0, 0.95)                                   # spike 10 nats above the bulk at T = 4
    add(rng.normal(0, 0.01, V), 5, 1.2, 0.93)                # near-flat: wide window
    add(rng.normal(0, 1.5, V) + 3000.0, 77, 1.0, 0.9)        # |A0| / T near 3,000: exact pass, coarse bf
    add(rng.normal(0, 1.5, V) + 30000.0, 78, 1.0, 0.9)       # |A0| / T beyond the binning guard: three passes
    logits, ids, T, P = _run(np.stack(rows), ids, Ts, Ps, dtype)
    print(f"case topp histogram edges {dtype}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


def test_topp_workload_scaled():
    """The top-p row model (V = 262,144 float32, T ~ U[0.3,1.2], P ~ U[0.8,0.95]) on a few requests."""
    w = wl.scaled(wl.WORKLOADS["topp_128x256_v262144_f32"], n_req=4, len_hi=6, len_lo=6)
    b = wl.make_batch(w, device="cpu")
    logits, ids, T, P = to_dev(b.logits, b.sampled_ids, b.temperature, b.top_p)
    print(f"case topp workload rows={b.n_rows}", flush=True)
    g = gpu_features(logits, ids, T, P)
    o = oracle_features(logits, ids, T, P)
    compare_features(g, o)
    assert (o["flags"] & pr.FLAG_OUTSIDE_NUCLEUS == 0).all()  # the sampler stays inside the nucleus


def test_topp_bf16_large_vocabulary():
    """The top-p row model on bf16 rows of the MLLM vocabulary (V = 151,936):
    the bf16 instantiation of the two-read method on realistic rows, every
    row against the oracle."""
    w = wl.scaled(wl.WORKLOADS["topp_128x256_v262144_f32"], n_req=6, len_hi=8, V=151936, dtype="bf16")
    b = wl.make_batch(w, device="cpu")
    logits, ids, T, P = to_dev(b.logits, b.sampled_ids, b.temperature, b.top_p)
    assert logits.dtype == torch.bfloat16
    print(f"case topp bf16 V=151936 rows={b.n_rows}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_flat_rows(dtype):
    """Flat and near-flat rows (sigma / T from 0.02 to 2, P from 0.5 to 0.99):
    the rows whose window many buckets reach, which take the float32 pass
    with its certified bound (and the float64 pass where the bound does not
    decide), against the oracle's exact cutoff."""
    V = 131072
    rng = np.random.default_rng(2024)
    n = 32
    sig = np.geomspace(0.02, 2.0, n)
    T = rng.uniform(0.5, 1.5, n)
    z = rng.normal(0, 1, (n, V)) * (sig * T)[:, None] + rng.uniform(-5, 5, (n, 1))
    P = rng.uniform(0.5, 0.99, n)
    ids = rng.integers(0, V, n)
    logits, ids, T, P = _run(z, ids, T, P, dtype)
    print(f"case topp flat rows V={V} {dtype}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_large_windows(dtype):
    """Windows of 513 to 4,096 logits, cut through their sub-buckets: a
    plateau of distinct values, a tie group of 1,500 at the crossing (its
    sub-bucket alone holds more than 512 logits and takes the workgroup
    sort), a window spanning fewer than 256 float steps (one value per
    sub-bucket), and one crossing zero (keys of both signs)."""
    V = 65536
    rng = np.random.default_rng(4096)
    rows, ids, Ps = [], [], []
    def add(z, P):
        pos = np.flatnonzero(z > -10)
        rows.append(z); ids.append(int(pos[len(pos) // 2])); Ps.append(P)
    for n, P in ((600, 0.6), (1500, 0.7), (3000, 0.8), (4000, 0.9)):
        z = np.full(V, -20.0)
        z[rng.choice(V, n, replace=False)] = rng.uniform(0.0, 1e-3, n)
        add(z, P)                                           # plateau of n distinct values
    z = np.full(V, -20.0)
    pos = rng.choice(V, 3000, replace=False)
    z[pos[:1500]] = 0.5
    z[pos[1500:]] = rng.uniform(0.49, 0.51, 1500)
    add(z, 0.5)                                             # 1,500 ties at the crossing
    z = np.full(V, -20.0)
    k = np.repeat(np.arange(200), 10)
    z[rng.choice(V, k.size, replace=False)] = 1.0 + k * 2.0 ** -23
    add(z, 0.6)                                             # 200 values one float step apart, 10 of each
    z = np.full(V, -20.0)
    z[rng.choice(V, 2500, replace=False)] = rng.uniform(-1e-3, 1e-3, 2500)
    add(z, 0.8)                                             # window across zero
    n = len(rows)
    logits, ids, T, P = _run(np.stack(rows), ids, np.ones(n), Ps, dtype)
    print(f"case topp large windows {dtype}", flush=True)
    g = gpu_features(logits, ids, T, P)
    compare_features(g, oracle_features(logits, ids, T, P))
    g2 = gpu_features(logits, ids, T, P)
    for key in g:
        assert np.array_equal(g[key].view(np.uint32), g2[key].view(np.uint32)), key


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_window_size_boundaries(dtype):
    """Windows at the limits of the one-wave cut's sizes (64, 128, 256, 512
    logits per wave, the sub-bucket cut above): a plateau of n values within
    one bin, the rest 20 nats below, the crossing inside the plateau."""
    V = 65536
    rng = np.random.default_rng(640)
    rows, ids, Ps = [], [], []
    for n in (1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513):
        z = np.full(V, -20.0)
        pos = rng.choice(V, n, replace=False)
        z[pos] = rng.uniform(0.0, 1e-4, n)
        rows.append(z); ids.append(int(pos[0])); Ps.append(0.5)
    n_rows = len(rows)
    logits, ids, T, P = _run(np.stack(rows), ids, np.ones(n_rows), Ps, dtype)
    print(f"case topp window size boundaries {dtype}", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


def test_topp_large_vocabulary():
    """A vocabulary of 2^20 + 3 (four times the largest workload's): random,
    flat and peaked rows against the oracle's exact cutoff."""
    V = (1 << 20) + 3
    rng = np.random.default_rng(20)
    rows = [rng.normal(0, 2, V), rng.normal(0, 0.01, V), rng.normal(0, 1, V)]
    rows[2][12345] = 40.0
    ids = [int(rng.integers(0, V)), 7, 12345]
    logits, ids, T, P = _run(np.stack(rows), ids, [0.8, 1.2, 1.0], [0.9, 0.93, 0.5])
    print("case topp V = 2^20 + 3", flush=True)
    compare_features(gpu_features(logits, ids, T, P), oracle_features(logits, ids, T, P))


def test_hardware_exp2_bound():
    """The float32 pass of the top-p kernel certifies its masses with a bound
    of 1e-7 on the relative error of the hardware exp2 (the constant
    kExp2RelErr) for arguments in [-100, 100] (its frame keeps t there):
    checked here over every float in [-126, 127]."""
    out = torch.zeros(2, dtype=torch.int64, device="cuda")
    st = wl.tools().prt_exp2_max_rel_err(-126.0, 127.0, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    w = out.cpu().numpy()
    err = float(w[:1].view(np.float64)[0])
    x = float(np.array([w[1]], dtype=np.int64).astype(np.uint32).view(np.float32)[0])
    print(f"case exp2 bound: largest relative error {err:.4e} (at x = {x:.9g})", flush=True)
    assert 0.0 < err <= 1.0e-7
    # a sub-range reports a largest error inside it, no larger than the whole range's
    out.zero_()
    assert wl.tools().prt_exp2_max_rel_err(-1.0, 1.0, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    w = out.cpu().numpy()
    e1 = float(w[:1].view(np.float64)[0])
    x1 = float(np.array([w[1]], dtype=np.int64).astype(np.uint32).view(np.float32)[0])
    assert -1.0 <= x1 <= 1.0 and 0.0 < e1 <= err


@pytest.mark.parametrize("dtype,V,offset", [(torch.float32, 65536, 0), (torch.float32, 65543, 1),
                                            (torch.bfloat16, 65536, 0), (torch.bfloat16, 70001, 3),
                                            (torch.float32, 98311, 1), (torch.bfloat16, 114699, 3)])
def test_topp_rows_over_several_workgroups(monkeypatch, dtype, V, offset):
    """Small batches of long rows, each over eight workgroups: every kind of
    row (flat, peaked, ties over the boundary, heavy ties, a distant maximum
    beyond the anchor's range, large |z| / T, masked logits, no nucleus,
    undefined, the sampled token outside), aligned and not, against the
    oracle; the same rows with one workgroup each agree in every whole
    number, and a second run is bit-identical."""
    rng = np.random.default_rng(V)
    n = 18
    s = np.concatenate([np.linspace(0.2, 6.0, 8), np.full(n - 8, 1.0)])[:, None]
    z = rng.normal(0, 1, (n, V)) * s
    z[np.arange(8), rng.integers(0, V, 8)] += rng.uniform(0, 15, 8)
    z[8] = 0.5                                   # every logit tied
    z[9] = np.round(z[9] * 4) / 4                # blocks of ties
    z[10, V - 1] = 120.0                         # far above the anchor
    z[11] += 6000.0                              # beyond the bins' accuracy
    z[12, rng.permutation(V)[:V // 2]] = -np.inf
    z[13, 7] = np.nan
    z[14] = -np.inf
    z[14, 9] = 1.0                               # one token
    z[15, V - 700:] += 40.0                      # more logits above the bins than the list holds
    ids = rng.integers(0, V, n)
    ids[:8:2] = np.argmax(z[:8:2], axis=1)
    T = rng.uniform(0.3, 1.2, n)
    P = rng.uniform(0.5, 0.98, n)
    P[16], T[17] = 1.0, -1.0
    wide = np.zeros((n, V + offset))
    wide[:, offset:] = z
    logits, ids, T, P = _run(wide, ids, T, P, dtype)
    logits = logits[:, offset:]
    print(f"case topp several workgroups V={V} offset={offset} {dtype}", flush=True)
    L = pr._abi.lib()
    assert L.pr_token_features_workspace_full(pr._dtype_code(logits), n, V, 1) > 0
    got = gpu_features(logits, ids, T, P)
    again = gpu_features(logits, ids, T, P)
    with monkeypatch.context() as m:
        m.setattr(L, "pr_token_features_workspace_full", lambda *a: 0)
        one = gpu_features(logits, ids, T, P)
    for k in got:
        assert np.array_equal(got[k].view(np.int32), again[k].view(np.int32)), k
    for k in ("rank", "argmax", "cutoff", "flags"):
        assert np.array_equal(got[k], one[k]), k
    ref = oracle_features(logits, ids, T, P)
    compare_features(got, ref)
    compare_features(one, ref)
    # the verifier input sequence: the K largest logits come from all parts
    off = torch.tensor([0, 5, n], dtype=torch.int32, device="cuda")
    for K in (1, 20, 32):
        X, f = pr.feature_sequence(logits, ids, T, off, top_p=P, top_k=K, features=True)
        with monkeypatch.context() as m:
            m.setattr(L, "pr_feature_sequence_workspace", lambda *a: 0)
            X1 = pr.feature_sequence(logits, ids, T, off, top_p=P, top_k=K)
        torch.cuda.synchronize()
        H = oseq.topk_entropy_batch(wl.to_host_raw(logits), "f32" if dtype == torch.float32 else "bf16",
                                    T.cpu().numpy(), P.cpu().numpy(), K)
        Xo = oseq.feature_sequence(ref, H, off.cpu().numpy())
        sure = ~ref["ambiguous"]
        for c in range(4):
            assert_floats(f"X[{c}] K={K}", X[:, c].cpu().numpy(), Xo[:, c], mask=sure)
            assert_floats(f"X[{c}] K={K}, one workgroup", X1[:, c].cpu().numpy(), Xo[:, c], mask=sure)
        for k in got:
            assert np.array_equal(f[k].cpu().numpy().view(np.int32), got[k].view(np.int32)), k


def test_topp_row_and_vocabulary_limits():
    """Either side of the batch sizes and vocabularies that spread their rows,
    at the workspace's exact size (nothing past it is written)."""
    L = pr._abi.lib()
    for dtype, n, V in ((torch.bfloat16, 32, 65536), (torch.bfloat16, 33, 65536), (torch.bfloat16, 2, 65535),
                        (torch.float32, 1, 131072), (torch.bfloat16, 128, 131072), (torch.bfloat16, 129, 131072)):
        full = int(L.pr_token_features_workspace_full(1 if dtype == torch.bfloat16 else 0, n, V, 1))
        assert (full > 0) == (n <= (128 if V >= 131072 else 32) and V >= 65536)
        g = torch.Generator(device="cuda").manual_seed(n)
        z = (torch.randn((n, V), generator=g, device="cuda") * 2.5).to(dtype)
        ids = torch.argmax(z.float(), 1).to(torch.int32)
        T, P = torch.full((n,), 0.8, device="cuda"), torch.full((n,), 0.9, device="cuda")
        buf = torch.full((full + 4096,), 0x7F, dtype=torch.uint8, device="cuda")
        print(f"case topp limits n={n} V={V} {dtype}", flush=True)
        f = pr.token_features(z, ids, T, P, workspace=buf[:max(full, 1)])
        torch.cuda.synchronize()
        assert bool((buf[full:] == 0x7F).all())
        rows = [0, n - 1]
        o = oracle_features(z, ids, T, P, rows)
        compare_features({k: v.cpu().numpy() for k, v in f.items()}, o, rows)


def test_token_features_leaves_the_workspace_alone_with_top_p():
    """pr_token_features asks for no workspace with top-p and does not touch one
    that it is given, whatever its alignment (a caller may pass one buffer to
    calls that overlap); pr_token_features_ws uses it, wants it aligned, and
    does without it when it is too small."""
    L = pr._abi.lib()
    n, V = 4, 70001
    g = torch.Generator(device="cuda").manual_seed(5)
    z = torch.randn((n, V), generator=g, device="cuda") * 2.5
    ids = torch.argmax(z, 1).to(torch.int32)
    T, P = torch.full((n,), 0.8, device="cuda"), torch.full((n,), 0.9, device="cuda")
    full = int(L.pr_token_features_workspace_full(pr._abi.PR_F32, n, V, 1))
    assert full > 0 and L.pr_token_features_workspace(pr._abi.PR_F32, n, V, 1) == 0
    buf = torch.full((full + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    ref = oracle_features(z, ids, T, P)

    def call(fn, shift, size):
        f = pr._alloc_features(n, z.device)
        st = fn(z.data_ptr(), pr._abi.PR_F32, n, V, V, ids.data_ptr(), T.data_ptr(), P.data_ptr(),
                C.byref(pr._features_struct(f)), buf.data_ptr() + shift, size, pr._stream_handle())
        torch.cuda.synchronize()
        if st == 0:
            compare_features({k: v.cpu().numpy() for k, v in f.items()}, ref)
        return st, bool((buf == 0xFF).all())

    print("case topp and the given workspace", flush=True)
    assert call(L.pr_token_features, 0, full) == (0, True)
    assert call(L.pr_token_features, 8, full) == (0, True)
    assert call(L.pr_token_features_ws, 0, full - 16) == (0, True)
    assert call(L.pr_token_features_ws, 8, full) == (pr._abi.PR_ERR_INVALID_ARG, True)
    assert call(L.pr_token_features_ws, 0, full) == (0, False)
    assert bool((buf[full:] == 0xFF).all())
    out = pr.token_features(z, ids, T, P, workspace=buf[8:])  # the binding does without a misaligned one
    compare_features({k: v.cpu().numpy() for k, v in out.items()}, ref)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topp_rows_masked_at_their_start(dtype):
    """Rows whose first 8,000 logits are masked, over several workgroups: what
    the oracle gives, in about the time of the same rows unmasked (the method
    for rows without an anchor takes three to five times as long)."""
    n, V = 16, 262144
    g = torch.Generator(device="cuda").manual_seed(17)
    z = (torch.randn((n, V), generator=g, device="cuda") * 2.5).to(dtype)
    T, P = torch.full((n,), 0.8, device="cuda"), torch.full((n,), 0.9, device="cuda")
    masked = z.clone()
    masked[:, :8000] = -math.inf
    print(f"case topp masked start {dtype}", flush=True)
    best = []
    for x in (z, masked):
        ids = torch.argmax(x.float(), 1).to(torch.int32)
        f = pr.token_features(x, ids, T, P)
        rows = [0, n - 1]
        compare_features({k: v.cpu().numpy() for k, v in f.items()}, oracle_features(x, ids, T, P, rows), rows)
        times = []
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                pr.token_features(x, ids, T, P)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times))
    assert best[1] < 2.0 * best[0], best


def test_sequence_row_and_vocabulary_limits():
    """Either side of the batches whose verifier input sequence spreads its
    rows: X against the oracle."""
    L = pr._abi.lib()
    for dtype, n, V, split in ((torch.bfloat16, 32, 65536, True), (torch.bfloat16, 33, 114687, False),
                               (torch.float32, 3, 127999, False), (torch.float32, 4, 65536, True),
                               (torch.bfloat16, 1, 128000, True), (torch.bfloat16, 64, 114688, True),
                               (torch.float32, 96, 131072, True), (torch.float32, 97, 131072, False),
                               (torch.bfloat16, 8, 65535, False), (torch.bfloat16, 128, 196608, True)):
        code = pr._abi.PR_BF16 if dtype == torch.bfloat16 else pr._abi.PR_F32
        assert (L.pr_feature_sequence_workspace(code, n, V, 1) > 0) == split
        g = torch.Generator(device="cuda").manual_seed(n)
        z = (torch.randn((n, V), generator=g, device="cuda") * 2.5).to(dtype)
        ids = torch.argmax(z.float(), 1).to(torch.int32)
        T, P = torch.full((n,), 0.8, device="cuda"), torch.full((n,), 0.9, device="cuda")
        off = torch.tensor([0, n], dtype=torch.int32, device="cuda")
        print(f"case sequence top-p limits n={n} V={V} {dtype}", flush=True)
        X = pr.feature_sequence(z, ids, T, off, top_p=P)[[0, n - 1]].cpu().numpy()
        rows = [0, n - 1]
        o = oracle_features(z, ids, T, P, rows)
        H = oseq.topk_entropy_batch(wl.to_host_raw(z[rows]), "f32" if dtype == torch.float32 else "bf16",
                                    T[rows].cpu().numpy(), P[rows].cpu().numpy(), 20)
        for c, ref in enumerate((o["logprob"], o["maxprob"], H, [1.0 / n, 1.0])):
            assert_floats(f"X[{c}] n={n} V={V}", X[:, c], -np.asarray(H) if c == 2 else np.asarray(ref, dtype=np.float64),
                          mask=~o["ambiguous"])

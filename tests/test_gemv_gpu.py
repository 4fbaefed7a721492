"""GPU parity of nmm_gemv / nmm_batched_gemv against the oracle, through the C ABI.

Floating-point cases must satisfy |y - y_ref| <= 4e-3 * sum_k |x_k W_kn| + 1e-6 elementwise;
integer-valued cases (every partial sum exact in fp32) must match bit for bit.  Sizes span
several panels, K-slices and ragged tails; the workload shapes are the full decode shapes.
"""
import numpy as np
import pytest
import torch

import oracle
import synthetic as syn
from gpu_util import assert_parity, dev16, host_bits

pytestmark = pytest.mark.gpu

nmm = pytest.importorskip("paper_2609_16009_amd")


def run_gemv(c: syn.GemvCase, path=None, ldy=None, fill=np.nan):
    path = nmm.NMM_PATH_AUTO if path is None else path
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    ldy = c.N if ldy is None else ldy
    y = torch.full((c.M, ldy), fill, dtype=torch.float32, device="cuda")
    nmm.nmm_gemv(x, W, y, N=c.N, path=path)
    torch.cuda.synchronize()
    return y


def check_case(c: syn.GemvCase, path=None):
    y = run_gemv(c, path)
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, K=c.K, N=c.N)
    return assert_parity(y, y_ref, a_ref, integer=c.integer, what=c.name)


@pytest.mark.parametrize("integer", [False, True])
def test_single_gemv_512_fp16(integer):
    check_case(syn.single_gemv_512(integer))


@pytest.mark.parametrize("integer", [False, True])
def test_down_projection_7168x2112(integer):
    check_case(syn.down_projection(integer))


def test_paper_matmul2_7168x576():
    check_case(syn.down_projection(n=576))


@pytest.mark.parametrize("M", [1, 2, 4, 8, 16, 32])
def test_uq_sweep_gemv_path(M):
    check_case(syn.uq_sweep(M), path=nmm.NMM_PATH_GEMV)


@pytest.mark.parametrize("M", [1, 16])
def test_uq_sweep_integer_exact(M):
    check_case(syn.uq_sweep(M, integer=True), path=nmm.NMM_PATH_GEMV)


def test_output_projection_16384x7168():
    check_case(syn.gemv_case(40, 1, 16384, 7168, syn.BF16, name="wo_16384x7168"))


RAGGED = [  # (M, K, N, dt, ldx, ldw)
    (3, 1021, 1031, syn.BF16, 1024, 1032),
    (1, 1, 1, syn.BF16, 8, 8),
    (5, 77, 3, syn.F16, 80, 8),
    (16, 4099, 520, syn.BF16, 4104, 520),
    (7, 9000, 4200, syn.F16, 9000, 4200),
    (1, 13, 8, syn.BF16, 16, 8),
    (2, 300, 64, syn.F16, 304, 64),
    (1, 33000, 24, syn.BF16, 33000, 24),
    (9, 1536, 3000, syn.BF16, 1536, 3000),
    (1, 2048, 8200, syn.BF16, 2048, 8200),
]


@pytest.mark.parametrize("M,K,N,dt,ldx,ldw", RAGGED)
def test_ragged_shapes_and_padding(M, K, N, dt, ldx, ldw):
    c = syn.gemv_case(1000 + M * K % 97, M, K, N, dt, ldx=ldx, ldw=ldw, name=f"ragged_{M}x{K}x{N}")
    check_case(c, path=nmm.NMM_PATH_GEMV)


@pytest.mark.parametrize("M,K,N,dt", [(3, 1021, 1031, syn.BF16), (16, 4099, 520, syn.F16),
                                      (1, 7168, 2112, syn.F16)])
def test_ragged_integer_exact(M, K, N, dt):
    c = syn.gemv_case(7, M, K, N, dt, integer=True, ldx=(K + 7) // 8 * 8, ldw=(N + 7) // 8 * 8,
                      name="ragged_int")
    check_case(c, path=nmm.NMM_PATH_GEMV)


@pytest.mark.parametrize("case", syn.random_gemv_shapes(), ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}_{c[6]}")
def test_random_shapes_integer_exact(case):
    # a seeded sweep over M, K, N, both 16-bit types, padded pitches and the three path choices
    # (the launch-bounds model checks the same cases): small integers, so every output is exact
    M, K, N, dt, ldx, ldw, path = case
    c = syn.gemv_case(500 + M + K % 97, M, K, N, dt, integer=True, ldx=ldx, ldw=ldw, name=f"random_{M}x{K}x{N}_{path}")
    check_case(c, path={"gemv": nmm.NMM_PATH_GEMV, "mfma": nmm.NMM_PATH_MFMA, "auto": nmm.NMM_PATH_AUTO}[path])


def test_largest_weight_extent_on_every_path():
    # one weight [65521, 16384] bf16 whose extent, 65521 * 16384 * 2 = 2^31 - 491,520 bytes, is just
    # under the 2^31-byte limit, so the 32-bit buffer offsets take their largest values.  As W
    # [65521, 16383] (padding column NaN) it feeds the GEMV (one row, every output) and the matrix
    # cores (16 rows, sampled columns); the same bytes as Wt [65521 rows, 16383 + 1] feed the
    # transposed path (sampled rows).  Values are small integers, so every sum is exact in fp32.
    K, N, ldw = 65521, 16383, 16384
    c = syn.large_int_case(61, 16, K, N, ldw)
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    rng = np.random.default_rng(5)
    y1 = torch.full((1, N), float("nan"), dtype=torch.float32, device="cuda")
    nmm.nmm_gemv(x[:1], W, y1, N=N, path=nmm.NMM_PATH_GEMV)
    y16 = torch.full((16, N), float("nan"), dtype=torch.float32, device="cuda")
    nmm.nmm_gemv(x, W, y16, N=N, path=nmm.NMM_PATH_MFMA)
    Kt, Nt = ldw - 1, K
    yt = torch.full((1, Nt), float("nan"), dtype=torch.float32, device="cuda")
    nmm.nmm_gemv_nt(x[:1, :Kt], W, yt, K=Kt)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.gemv(c.x[:1], c.W, c.dt, K=K, N=N)
    assert_parity(y1, y_ref, a_ref, integer=True, what="GEMV at the largest extent")
    cols = np.unique(np.r_[0, 1, 127, 128, 8191, 8192, N - 129, N - 2, N - 1, rng.choice(N, 119, replace=False)])
    y_ref, a_ref = oracle.gemv(c.x, np.ascontiguousarray(c.W[:, cols]), c.dt, K=K, N=len(cols))
    assert_parity(y16[:, cols], y_ref, a_ref, integer=True, what="MFMA at the largest extent")
    rows = np.unique(np.r_[0, 1, 31, 32, Nt // 2, Nt - 33, Nt - 2, Nt - 1, rng.choice(Nt, 120, replace=False)])
    Ws = np.ascontiguousarray(c.W[rows, :Kt].T)           # [Kt, len(rows)]: the sampled rows of Wt as W
    y_ref, a_ref = oracle.gemv(c.x[:1], Ws, c.dt, K=Kt, N=len(rows))
    assert_parity(yt[:, rows], y_ref, a_ref, integer=True, what="transposed path at the largest extent")


def test_output_padding_untouched():
    c = syn.gemv_case(3, 2, 500, 70, syn.BF16, ldx=504, ldw=72)
    y = run_gemv(c, ldy=80, fill=-7.0)
    assert torch.all(y[:, 70:] == -7.0)
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, N=70)
    assert_parity(y[:, :70], y_ref, a_ref)


def test_deterministic_and_workspace_reuse():
    big = syn.down_projection()
    small = syn.gemv_case(9, 1, 4000, 1000, syn.BF16)
    ws = nmm.Workspace()
    outs = []
    for c in (big, small, big, small):
        x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
        y = torch.empty((1, c.N), dtype=torch.float32, device="cuda")
        nmm.nmm_gemv(x, W, y, workspace=ws)
        torch.cuda.synchronize()
        outs.append(y.cpu())
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[3])
    y_ref, a_ref = oracle.gemv(small.x, small.W, small.dt)
    assert_parity(outs[3], y_ref, a_ref)
    # every arrival counter (the workspace's first 64 KiB) is back at zero after the calls
    tickets = ws.buf[:65536].view(torch.int32)
    assert int(tickets.abs().sum()) == 0


@pytest.mark.parametrize("K,N", [(7168, 2112), (16384, 7168), (7168, 576)], ids=["down", "w_o", "matmul2"])
def test_split_k_soak_bit_identical(K, N):
    # 1000 launches of a split-K shape on one workspace: every result equals the first bit for
    # bit (the gather sums the slices in a fixed order, whichever XCD finishes first), and the
    # arrival counters are back at zero after the last
    c = syn.gemv_case(50, 1, K, N, syn.BF16, name=f"soak_{K}x{N}")
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    ws = nmm.Workspace()
    assert nmm.nmm_gemv_plan(1, K, N, syn.BF16, nmm.NMM_PATH_AUTO)["split_k_full"] > 1
    ref = torch.empty((1, N), dtype=torch.float32, device="cuda")
    nmm.nmm_gemv(x, W, ref, workspace=ws)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt)
    assert_parity(ref, y_ref, a_ref, what=c.name)
    ys = torch.empty((20, 1, N), dtype=torch.float32, device="cuda")
    for batch in range(50):
        ys.fill_(float("nan"))
        for i in range(20):
            nmm.nmm_gemv(x, W, ys[i], workspace=ws)
        same = (ys == ref).all(dim=2).view(-1)
        if not bool(same.all()):
            first = batch * 20 + int((~same).nonzero()[0])
            raise AssertionError(f"{c.name}: launch {first} differs from the first result")
    assert int(ws.buf[:65536].view(torch.int32).abs().sum()) == 0


def test_k_zero_writes_zeros_and_empty_is_noop():
    x = torch.zeros((2, 8), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((1, 16), dtype=torch.bfloat16, device="cuda")
    y = torch.full((2, 16), 5.0, device="cuda")
    st = nmm.lib().nmm_gemv(2, 0, 16, nmm.NMM_BF16, x.data_ptr(), 8, W.data_ptr(), 16, y.data_ptr(), 16,
                            0, None, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == nmm.NMM_OK and torch.all(y == 0)
    y.fill_(5.0)
    st = nmm.lib().nmm_gemv(0, 8, 16, nmm.NMM_BF16, x.data_ptr(), 8, W.data_ptr(), 16, y.data_ptr(), 16,
                            0, None, 0, None)
    torch.cuda.synchronize()
    assert st == nmm.NMM_OK and torch.all(y == 5.0)


def test_invalid_call_enqueues_nothing():
    c = syn.gemv_case(5, 1, 256, 256, syn.BF16)
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    y = torch.full((1, 256), 3.0, device="cuda")
    st = nmm.lib().nmm_gemv(1, 256, 256, nmm.NMM_BF16, x.data_ptr(), 256, W.data_ptr() + 2, 256,
                            y.data_ptr(), 256, 0, None, 0, None)
    torch.cuda.synchronize()
    assert st == nmm.NMM_ERR_ALIGN and torch.all(y == 3.0)


def _loaded_hip_runtime():
    """The HIP runtime library this process has loaded (the one libnmm's calls go to)."""
    import ctypes
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64.so" in line}
    assert paths, "no HIP runtime loaded"
    return ctypes.CDLL(sorted(paths)[0])


def test_hip_error_reaches_the_caller_as_nmm_err_hip():
    # NMM_ERR_HIP reports what the HIP runtime says after the launch: here an error left unread
    # by an earlier runtime call on this thread (an invalid device ordinal, refused on the host;
    # nothing reaches the GPU), which the call reports once and so clears
    c = syn.gemv_case(5, 1, 256, 256, syn.BF16)
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    y = torch.empty((1, 256), device="cuda")
    torch.cuda.synchronize()
    hip = _loaded_hip_runtime()
    assert hip.hipSetDevice(1 << 20) != 0
    args = (1, 256, 256, nmm.NMM_BF16, x.data_ptr(), 256, W.data_ptr(), 256, y.data_ptr(), 256, 0, None, 0, None)
    assert nmm.lib().nmm_gemv(*args) == nmm.NMM_ERR_HIP
    torch.cuda.synchronize()
    assert nmm.lib().nmm_gemv(*args) == nmm.NMM_OK
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt)
    assert_parity(y, y_ref, a_ref)


@pytest.mark.parametrize("M", [1, 2])
@pytest.mark.parametrize("K,N", [(512, 700), (513, 700), (700, 20000), (3000, 3000), (16384, 2500), (1100, 9001), (4099, 5003),
                                 (7168, 1031), (6000, 9001), (130, 33000)])
def test_narrow_plans_integer_exact(M, K, N):
    # one- and two-row plans: unsplit and split, panels of 8, 16 and 32 chunks, items in XCD runs (rows that
    # start inside a line) and in plain order (ldw a multiple of 64), ragged last panels
    for ldw in ((N + 7) // 8 * 8, (N + 63) // 64 * 64):
        c = syn.gemv_case(M + K % 71, M, K, N, syn.BF16, integer=True, ldx=(K + 7) // 8 * 8, ldw=ldw)
        y = torch.full((M, N + 1), float("nan"), dtype=torch.float32, device="cuda")
        nmm.nmm_gemv(dev16(c.x, c.dt), dev16(c.W, c.dt), y, N=N, path=nmm.NMM_PATH_GEMV)
        torch.cuda.synchronize()
        y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, K=K, N=N)
        assert_parity(y[:, :N], y_ref, a_ref, integer=True, what=f"narrow {M}x{K}x{N} ld {ldw}")
        assert torch.isnan(y[:, N:]).all()


@pytest.mark.parametrize("M", [1, 2])
@pytest.mark.parametrize("K,N", [(64, 66001), (65, 17000), (300, 70000), (200, 131000), (520, 33000), (800, 65600)])
def test_wide_rows_integer_exact(M, K, N):
    # panels of 64, 16, 16, 64, 32 and (two slices and a last panel of 8 chunks) 64 chunks, all off the tile edges
    c = syn.gemv_case(K + N, M, K, N, syn.BF16, integer=True, ldx=(K + 7) // 8 * 8, ldw=(N + 7) // 8 * 8)
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, K=K, N=N)
    y = torch.full((M, N + 3), float("nan"), dtype=torch.float32, device="cuda")
    nmm.nmm_gemv(dev16(c.x, c.dt), dev16(c.W, c.dt), y, N=N, path=nmm.NMM_PATH_GEMV)
    torch.cuda.synchronize()
    assert_parity(y[:, :N], y_ref, a_ref, integer=True, what=f"{M}x{K}x{N}")
    assert torch.isnan(y[:, N:]).all(), "columns past N were written"


def test_infinity_propagates_to_its_column_only():
    c = syn.gemv_case(6, 1, 3000, 700, syn.BF16, ldw=704)
    W = c.W.copy()
    W[1234, 321] = 0x7F80          # +inf
    x = c.x.copy()
    x[0, 1234] = 0x3F80            # 1.0
    y = run_gemv(syn.GemvCase(1, 3000, 700, syn.BF16, x, W, name="inf"))
    y = y.cpu().numpy()[0]
    assert np.isposinf(y[321])
    mask = np.ones(700, bool)
    mask[321] = False
    assert np.isfinite(y[mask]).all()


def test_a_workspace_grows_when_a_call_asks_and_a_given_buffer_does_not():
    # the call is tried on the workspace as it stands: a fresh or outgrown Workspace is grown and the call
    # repeated, on the caller's stream; a tensor that is too small stays refused, with y untouched
    s = torch.cuda.Stream()
    ws = nmm.Workspace()
    for M, K, N in ((1, 7168, 576), (4, 7168, 2112), (1, 512, 512), (16, 16384, 7168)):
        c = syn.gemv_case(40 + M, M, K, N, syn.BF16, integer=True)
        x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
        y = torch.zeros((M, N), device="cuda")
        torch.cuda.synchronize()
        need = nmm.nmm_gemv_workspace_size(M, K, N)
        nmm.nmm_gemv(x, W, y, workspace=ws, stream=s)
        s.synchronize()
        y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt)
        assert_parity(y, y_ref, a_ref, integer=True)
        assert need == 0 or ws.buf.numel() >= need and ws.held == (ws.buf.data_ptr(), ws.buf.numel())
        if need:
            with pytest.raises(nmm.NmmError) as e:
                nmm.nmm_gemv(x, W, y.zero_(), workspace=torch.zeros(need // 2, dtype=torch.uint8, device="cuda"))
            torch.cuda.synchronize()
            assert e.value.status == nmm.NMM_ERR_WORKSPACE and not y.any()


# ------------------------------------------------------------------ batched (per-head)

def test_absorbed_heads_two_steps():
    h = syn.absorbed_heads()
    q = dev16(h.q_nope, h.dt)
    uk, uv = dev16(h.w_uk, h.dt), dev16(h.w_uv, h.dt)
    lat = torch.empty((128, 1, 512), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(q, uk, lat)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(h.q_nope, h.w_uk, h.dt)
    assert_parity(lat, y_ref, a_ref, what="q_nope . W_UK")
    # step 2 consumes the GPU's step-1 result rounded to bf16 (ties to even)
    lat_bits = oracle.round_bf16(lat.cpu().numpy())
    o = torch.empty((128, 1, 128), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(dev16(lat_bits, h.dt), uv, o)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(lat_bits, h.w_uv, h.dt)
    assert_parity(o, y_ref, a_ref, what="latent . W_UV")


def test_absorbed_heads_integer_exact():
    h = syn.absorbed_heads(integer=True)
    lat = torch.empty((128, 1, 512), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(dev16(h.q_nope, h.dt), dev16(h.w_uk, h.dt), lat)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(h.q_nope, h.w_uk, h.dt)
    assert_parity(lat, y_ref, a_ref, integer=True, what="int q_nope . W_UK")


def test_batched_strided_query_slice():
    # q_nope is the first 128 of each head's 192 columns: a strided view, stride 192
    rng = np.random.default_rng(8)
    q_full = syn.normal_bits(rng, (128, 1, 192), 1.0, syn.BF16)
    h = syn.absorbed_heads()
    qd = dev16(q_full, syn.BF16)[:, :, :128]
    lat = torch.empty((128, 1, 512), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(qd, dev16(h.w_uk, h.dt), lat)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(np.ascontiguousarray(q_full[:, :, :128]), h.w_uk, h.dt)
    assert_parity(lat, y_ref, a_ref, what="strided q_nope")


@pytest.mark.parametrize("B,M,K,N", [(3, 2, 1000, 72), (128, 1, 512, 128), (5, 16, 96, 1000), (2, 1, 20000, 40)])
def test_batched_ragged(B, M, K, N):
    rng = np.random.default_rng(B * 1000 + K)
    x = syn.normal_bits(rng, (B, M, K), 1.0, syn.BF16)
    W = syn.normal_bits(rng, (B, K, N), 1.0 / np.sqrt(K), syn.BF16)
    y = torch.empty((B, M, N), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(dev16(x, syn.BF16), dev16(W, syn.BF16), y, path=nmm.NMM_PATH_GEMV)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(x, W, syn.BF16)
    assert_parity(y, y_ref, a_ref, what=f"batched {B}x{M}x{K}x{N}")


@pytest.mark.parametrize("case", syn.random_batched_shapes(), ids=lambda c: "x".join(map(str, c)))
def test_batched_random_shapes_integer_exact(case):
    # a seeded sweep (the launch-bounds model checks the same cases): small integers, so every
    # output of every batch entry is exact
    B, M, K, N = case
    rng = np.random.default_rng(B * 7919 + K + N)
    x = syn.int_bits(rng, (B, M, K), syn.BF16)
    W = syn.int_bits(rng, (B, K, N), syn.BF16)
    y = torch.full((B, M, N), float("nan"), dtype=torch.float32, device="cuda")
    nmm.nmm_batched_gemv(dev16(x, syn.BF16), dev16(W, syn.BF16), y, path=nmm.NMM_PATH_GEMV)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.batched_gemv(x, W, syn.BF16)
    assert_parity(y, y_ref, a_ref, integer=True, what=f"batched {B}x{M}x{K}x{N}")


@pytest.mark.parametrize("B,M", [(2, 1), (300, 1), (3, 2), (2, 15), (3, 16), (2, 17), (2, 33)])
@pytest.mark.parametrize("K,N", [(1, 1), (31, 63), (128, 64), (129, 65), (256, 700), (513, 128), (2048, 9)])
def test_batched_matrix_core_edges_integer_exact(B, M, K, N):
    # AUTO's batched matrix-core launch at the edges of its row, column and K tiles: NaN in every
    # padding value, outputs on and off 16-byte rows, fp32 and bf16 (either tie rule), alone and together
    rng = np.random.default_rng(B * 31 + M * 7 + K + N)
    K8, N8 = (K + 7) // 8 * 8, (N + 7) // 8 * 8
    for dt, ldy in ((syn.BF16, N8 + 4), (syn.F16, N + 1)):
        x = np.stack([syn.padded(a, K8) for a in syn.int_bits(rng, (B, M, K), dt)])
        W = np.stack([syn.padded(a, N8 + 8) for a in syn.int_bits(rng, (B, K, N), dt)])
        xd, Wd = dev16(x, dt), dev16(W, dt)
        y_ref, a_ref = oracle.batched_gemv(x, W, dt, N=N)
        y = torch.full((B, M, ldy), float("nan"), dtype=torch.float32, device="cuda")
        nmm.nmm_batched_gemv(xd, Wd, y, N=N)
        yb = torch.full((B, M, ldy), float("nan"), dtype=torch.bfloat16, device="cuda")
        y2 = torch.empty((B, M, N), dtype=torch.float32, device="cuda")
        nmm.nmm_batched_gemv_bf16(xd, Wd, yb, y=y2, N=N, round=nmm.NMM_ROUND_AWAY)
        yc = torch.empty((B, M, N), dtype=torch.bfloat16, device="cuda")
        nmm.nmm_batched_gemv_bf16(xd, Wd, yc, N=N)
        torch.cuda.synchronize()
        assert_parity(y[:, :, :N], y_ref, a_ref, integer=True, what=f"heads {B}x{M}x{K}x{N}")
        assert torch.equal(y2, y[:, :, :N]) and torch.equal(yc, y2.to(torch.bfloat16))
        assert torch.isnan(y[:, :, N:]).all() and torch.isnan(yb[:, :, N:]).all(), "columns past N were written"
        away = oracle.round_bf16(y2.cpu().numpy(), mode=1)
        assert np.array_equal(yb[:, :, :N].contiguous().view(torch.int16).cpu().numpy().view(np.uint16), away)


@pytest.mark.parametrize("K", [128, 100, 1024])
def test_batched_matrix_cores_agree_with_the_stream(K):
    # AUTO against the streaming form over strided slices, a broadcast weight and both 16-bit types
    g = torch.Generator(device="cuda").manual_seed(K)
    for dt in (torch.bfloat16, torch.float16):
        x = torch.randn((6, 5, 2 * K + 56), generator=g, device="cuda").to(dt)[:, 1:4, :K]
        W = (torch.randn((1, K, 208), generator=g, device="cuda") / K ** 0.5).to(dt).expand(6, K, 208)
        a, b = (torch.empty((6, 3, 200), device="cuda") for _ in range(2))
        nmm.nmm_batched_gemv(x, W, a, N=200)
        nmm.nmm_batched_gemv(x, W, b, N=200, path=nmm.NMM_PATH_GEMV)
        torch.cuda.synchronize()
        # both sum exact products in fp32 or wider: K roundings of 2^-24 at most, against sums near 1
        assert (a - b).abs().max().item() < K * 2.0 ** -24 * 8


# ------------------------------------------------------------------ matrix-core path

@pytest.mark.parametrize("M", [3, 15, 16, 17, 31, 33])
@pytest.mark.parametrize("K,N", [(512, 512), (1024, 2560), (4096, 5003), (2049, 16700)])
def test_mfma_slices_integer_exact(M, K, N):
    # slice counts that are no power of two, the gather of the real rows of a 16- or 32-row tile, and
    # output rows on and off 16 bytes
    c = syn.gemv_case(M + K % 89, M, K, N, syn.BF16, integer=True, ldx=(K + 7) // 8 * 8, ldw=(N + 7) // 8 * 8)
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, K=K, N=N)
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    for ldy in ((N + 3) // 4 * 4 + 4, N + 1):
        y = torch.full((M, ldy), float("nan"), dtype=torch.float32, device="cuda")
        nmm.nmm_gemv(x, W, y, N=N)
        torch.cuda.synchronize()
        assert_parity(y[:, :N], y_ref, a_ref, integer=True, what=f"slices {M}x{K}x{N}")
        if ldy > N:
            assert torch.isnan(y[:, N:]).all(), "columns past N were written"


@pytest.mark.parametrize("M", [3, 16, 17, 33])
@pytest.mark.parametrize("K,N", [(130, 33335), (70, 33336), (1024, 9001), (520, 520)])
def test_mfma_output_forms_integer_exact(M, K, N):
    # one slice (261 panels), three and eight; fp32 rows and bf16 rows on and off the boundary of their wide
    # stores, together and alone; the columns past N keep what they held
    c = syn.gemv_case(M + K, M, K, N, syn.BF16, integer=True, ldx=(K + 7) // 8 * 8, ldw=(N + 7) // 8 * 8)
    y_ref, a_ref = oracle.gemv(c.x, c.W, c.dt, K=K, N=N)
    b_ref = oracle.round_bf16(y_ref.astype(np.float32))
    x, W = dev16(c.x, c.dt), dev16(c.W, c.dt)
    on, off = (N + 3) // 4 * 4 + 4, (N + 3) // 4 * 4 + 5
    for ldy, ldyb in ((on, on), (off, on), (on, off), (off, off), (None, on), (None, off), (off, None)):
        y = torch.full((M, ldy), float("nan"), dtype=torch.float32, device="cuda") if ldy else None
        yb = torch.full((M, ldyb), float("nan"), dtype=torch.bfloat16, device="cuda") if ldyb else None
        if yb is None:
            nmm.nmm_gemv(x, W, y, N=N)
        else:
            nmm.nmm_gemv_bf16(x, W, yb, N=N, y=y)
        torch.cuda.synchronize()
        if y is not None:
            assert_parity(y[:, :N], y_ref, a_ref, integer=True, what=f"fp32 rows {M}x{K}x{N}, ldy {ldy}, ldyb {ldyb}")
            assert torch.isnan(y[:, N:]).all(), "columns past N were written"
        if yb is not None:
            assert np.array_equal(host_bits(yb)[:, :N], b_ref), f"bf16 rows {M}x{K}x{N}, ldy {ldy}, ldyb {ldyb}"
            assert torch.isnan(yb[:, N:]).all(), "columns past N were written"


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 8, 16, 17, 32])
def test_uq_sweep_mfma_path(M):
    check_case(syn.uq_sweep(min(M, 32)) if M <= 32 else None, path=nmm.NMM_PATH_MFMA)


@pytest.mark.parametrize("M", [4, 32])
def test_uq_sweep_mfma_integer_exact(M):
    check_case(syn.uq_sweep(M, integer=True), path=nmm.NMM_PATH_MFMA)


@pytest.mark.parametrize("M,K,N,dt,ldx,ldw", [(5, 1021, 1031, syn.BF16, 1024, 1032), (33, 4099, 520, syn.F16, 4104, 520),
                                              (8, 100, 8, syn.BF16, 104, 8), (32, 20000, 300, syn.F16, 20000, 304),
                                              (17, 16384, 7168, syn.BF16, 16384, 7168)])
def test_mfma_ragged(M, K, N, dt, ldx, ldw):
    c = syn.gemv_case(77 + M, M, K, N, dt, ldx=ldx, ldw=ldw, name=f"mfma_{M}x{K}x{N}")
    check_case(c, path=nmm.NMM_PATH_MFMA)
    ci = syn.gemv_case(78 + M, M, K, N, dt, integer=True, ldx=ldx, ldw=ldw, name=f"mfma_int_{M}x{K}x{N}")
    check_case(ci, path=nmm.NMM_PATH_MFMA)


def test_auto_path_switches_at_crossover():
    # one row streams; W_UQ's matrix-core plan has a single K-slice, so two rows take the matrix
    # cores there, while W_O's (split K) keeps the streaming GEMV at two rows
    assert nmm.nmm_gemv_plan(1, 1536, 24576)["path"] == nmm.NMM_PATH_GEMV
    assert nmm.nmm_gemv_plan(2, 16384, 7168)["path"] == nmm.NMM_PATH_GEMV
    for M in (2, 3, 4, 16, 32):
        assert nmm.nmm_gemv_plan(M, 1536, 24576)["path"] == nmm.NMM_PATH_MFMA
    assert nmm.nmm_gemv_plan(16, 128, 512, batch=8)["path"] == nmm.NMM_PATH_GEMV


@pytest.mark.parametrize("M", [17, 20])
def test_remnant_split_on_two_streams(M):
    # the paper's Condition 4 split: rows [0, 16q) on the matrix cores and the remnant rows on
    # the streaming GEMV, concurrently on two streams into one y; both parts meet the fp32 bar
    c = syn.uq_sweep(32)
    q16 = M // 16 * 16
    x, W = dev16(c.x[:M], syn.BF16), dev16(c.W, syn.BF16)
    y = torch.full((M, c.N), float("nan"), dtype=torch.float32, device="cuda")
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    start = torch.cuda.Event()
    start.record()
    sa.wait_event(start)
    sb.wait_event(start)
    nmm.nmm_gemv(x[:q16], W, y[:q16], path=nmm.NMM_PATH_MFMA, workspace=nmm.Workspace(), stream=sa)
    nmm.nmm_gemv(x[q16:], W, y[q16:], path=nmm.NMM_PATH_GEMV, workspace=nmm.Workspace(), stream=sb)
    torch.cuda.synchronize()
    y_ref, a_ref = oracle.gemv(c.x[:M], c.W, syn.BF16)
    assert_parity(y, y_ref, a_ref, what=f"remnant split M={M}")

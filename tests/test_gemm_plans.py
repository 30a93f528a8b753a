"""GEMM plans: the planner's rules (host) and every kernel, tile and epilogue a plan can name,
forced at the edges of its tiles (GPU, against fp64 products of the same operands)."""

import ctypes
import math
import random

import pytest
import torch

F32, BF16, F16 = 0, 1, 2
BIAS_N, GELU, RES, BIAS_M, HILO, PART = range(6)
TILE256, TILE128, MID, SKINNY = range(4)
P, I, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64


class Desc(ctypes.Structure):       # kraken::GemmDesc
    _fields_ = [("dt", I), ("epi", I), ("A", P), ("B", P), ("C", P), ("bias", P), ("R", P),
                ("M", I), ("N", I), ("K", I), ("lda", I), ("ldb", I), ("ldc", I), ("sA", L),
                ("sB", L), ("sC", L), ("sR", L), ("sBias", L), ("batch", I), ("kgroups", I),
                ("gA", L), ("gB", L), ("gBmod", I), ("splits", I), ("sPlane", L),
                ("gA2", L), ("qkv", P), ("ovf", P)]


class Plan(ctypes.Structure):       # kraken::GemmPlan
    _fields_ = [("kind", I), ("nb", I), ("splits", I), ("waves", I)]


def _lib():
    from paper_2408_07802_amd import kraken
    return kraken.lib()


def plan(dt, epi, M, N, K, kgroups, batch, part, own_sum=False, terms=1):
    f = getattr(_lib(), "_ZN6kraken9plan_gemmENS_5DTypeEiiiiiiilb")
    f.argtypes, f.restype = [I] * 8 + [L, ctypes.c_bool], Plan
    return f(dt, epi, M, N, K, kgroups, terms, batch, part, own_sum)


def few_row_forms(dt, M):
    """(column blocks, waves) of the few-row kernels that are built for M rows."""
    if dt == F32:
        return [(1, 16)] if M <= 16 else [(1, 8)] if M <= 64 else []
    return [(1, 4), (1, 8), (2, 8)] if M <= 16 else [(1, 8)] if M <= 32 else []


def test_every_few_row_form_is_planned():
    # each form that is built is the plan of some shape, and no plan names another
    rng, seen = random.Random(11), {}
    for _ in range(40000):
        dt, M = rng.choice([F32, F16]), rng.randint(1, 64)
        N, K = 4 * rng.randint(1, 8192), 64 * rng.randint(1, 256)
        b, terms = rng.choice([1, 2, 4, 8]), rng.choice([1, 2])
        p = plan(dt, RES, M, N, K, 1, b, rng.choice([0, 1 << 40]), terms=terms)
        if p.kind == SKINNY:
            rows = 16 if M <= 16 else 32 if M <= 32 else 64
            assert (p.nb, p.waves) in few_row_forms(dt, M)
            seen.setdefault((dt, rows), set()).add((p.nb, p.waves))
    assert seen == {(dt, r): set(few_row_forms(dt, r)) for dt, r in
                    [(F32, 16), (F32, 32), (F32, 64), (F16, 16), (F16, 32)]}


def test_plans_stay_within_their_limits():
    rng = random.Random(3)
    for _ in range(4000):
        dt = rng.choice([F32, BF16, F16])
        M = int(math.exp(rng.uniform(0, math.log(20000))))
        N, K = 4 * rng.randint(1, 4096), 64 * rng.randint(1, 256)
        g, b = rng.choice([1, 1, 2, 16]), rng.choice([1, 2, 4, 8])
        part = rng.choice([0, M * N * b, 5 * M * N * b, 1 << 40])
        epi = rng.choice([RES, RES, PART])
        p = plan(dt, epi, M, N, K, g, b, part, rng.random() < 0.5)
        assert p.kind != SKINNY or M <= 64
        assert p.kind == SKINNY or M > (64 if dt == F32 else 16)
        assert p.kind != SKINNY or (p.nb, p.waves) in few_row_forms(dt, M)
        assert p.kind != MID or 1 <= p.nb <= 6
        slices = K // (32 if dt == F32 else 64) * g
        assert 1 <= p.splits <= 8 and (p.splits == 1 or (2 if dt == F32 else 8) * p.splits <= slices)
        assert p.splits == 1 or p.splits * M * N * b <= part


@pytest.mark.parametrize("dt,terms", [(F32, 1), (F16, 1), (F16, 2)])
def test_few_row_splits_leave_every_wave_a_batch_of_loads(dt, terms):
    # the splits of a W_concat (own_sum), in the steps that the kernel really walks: 8 loads of
    # A for every wave, whichever number of terms a step loads
    rng, split = random.Random(5), 0
    for _ in range(3000):
        M, N, d = rng.choice([1, 2, 7, 16]), rng.choice([1, 2, 4, 8]), 64 * rng.randint(2, 40)
        p = plan(dt, RES, M, d, d, N, 1, 1 << 26, True, terms=terms)
        assert p.kind == SKINNY
        steps = N * d // (16 if dt == F32 else 32)
        if p.splits > 1:
            split += 1
            assert steps * terms // (p.splits * p.waves) >= 8, (M, N, d, p.splits, p.waves)
    assert split > 100


def test_benchmark_layer_is_whole_at_4096_and_8192_rows():
    # the benchmark layer at these two lengths alone: whole reductions, so the longer prompt's
    # rows have the bits of the shorter one's (which a GPU test compares)
    for M in (4096, 8192):
        for N, K in ((4096, 2048), (2048, 2048), (8192, 2048), (2048, 8192)):
            assert plan(F16, RES, M, N, K, 1, 8, 1 << 26).splits == 1
        assert plan(F16, RES, M, 2048, 2048, 8, 1, 1 << 26, True, terms=2).splits == 1  # W_concat


def test_sums_with_a_launch_of_their_own_stay_whole_from_512_tiles():
    # W_concat (N sub-layers of width d), from the row count on that the planner's comment names
    for N, d, rows in ((8, 2048, 3969), (4, 1280, 6529), (4, 1024, 8065)):
        for M in [rows, rows + 1] + [random.Random(d).randint(rows, 20000) for _ in range(50)]:
            assert plan(F16, RES, M, d, d, N, 1, 1 << 26, True, terms=2).splits == 1, (M, d)
    # and no promise below it, nor for a plane that the next kernel sums
    assert plan(F16, RES, 4096, 1280, 1280, 4, 1, 1 << 26, True, terms=2).splits == 3
    assert plan(F16, RES, 4096, 1024, 1024, 4, 1, 1 << 26, True, terms=2).splits == 4
    assert plan(F16, RES, 3584, 2048, 2048, 8, 1, 1 << 26, True, terms=2).splits > 1
    assert plan(F16, RES, 9000, 2048, 8192, 1, 1, 1 << 26).splits == 2


@pytest.mark.parametrize("empty", ["M", "N", "batch", "kgroups"])
def test_an_empty_product_needs_no_plan(empty):
    # (the planner divides by tile counts; nothing is launched)
    f = getattr(_lib(), "_ZN6kraken11launch_gemmERKNS_8GemmDescEP12ihipStream_t")
    f.restype = I
    for dt in (F32, F16):
        for M in (8, 100):
            d = Desc(dt=dt, epi=BIAS_N, M=M, N=64, K=64, lda=64, ldb=64, ldc=64, batch=1, kgroups=1,
                     gBmod=1)
            setattr(d, empty, 0)
            assert f(ctypes.byref(d), P(None)) == 0


def test_models_allocate_the_planes_that_their_plans_ask_for():
    from paper_2408_07802_amd import kraken
    f = getattr(_lib(), "_ZN6kraken19partial_plane_elemsEPK13kraken_configi")
    f.argtypes, f.restype = [P, I], L

    def elems(cfg, T):                  # of a pass over T rows; T = 0: of the model
        c = cfg.c_struct()
        return f(ctypes.addressof(c), T)

    rng, split = random.Random(7), 0
    for _ in range(300):
        arch = rng.choice(["kraken", "gpt", "parallel"])
        hd, heads = rng.choice([32, 64, 128]), 2 * rng.randint(1, 16)
        cfg = kraken.Config(
            n_sub=rng.choice([1, 2, 4, 8]) if arch == "kraken" else 1, n_layers=rng.choice([1, 2]),
            d_model=hd * heads - rng.choice([0, 0, 20]), n_heads=heads, head_dim=hd,
            d_ff=hd * heads * rng.choice([1, 2, 4]), arch=arch, dtype=rng.choice(["f16", "f32"]),
            max_tokens=int(math.exp(rng.uniform(0, math.log(20000)))))
        room, T = elems(cfg, 0), cfg.max_tokens
        assert room <= 64 << 20
        need = [elems(cfg, t) for t in [T] + [rng.randint(1, T) for _ in range(40)]]
        assert max(need) <= room, cfg
        split += max(need) > 0
    assert split > 100
    # a small model does not pay for planes that none of its plans can have (8 planes of the
    # widest result would be 256 MB)
    small = kraken.Config(n_sub=4, n_layers=1, d_model=1024, n_heads=16, d_ff=4096,
                          max_tokens=2048, dtype="bf16", compute="f16")
    assert elems(small, 0) * 4 <= 32 << 20


# (M, N, K, batch, K splits): one row past and short of tiles of 128 and 256, column counts
# that are no multiple of a tile or of 4, splits of unequal length, a single slice
SHAPES = [(65, 96, 64, 1, 1), (127, 130, 192, 2, 3), (128, 160, 128, 1, 2), (129, 257, 320, 2, 5),
          (255, 64, 640, 1, 4), (257, 320, 512, 2, 8), (300, 33, 448, 3, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("epi", [BIAS_N, GELU, RES, BIAS_M, HILO, PART])
@pytest.mark.parametrize("dt", [F32, BF16, F16])
def test_every_plan_at_tile_edges(dt, epi):
    if epi == HILO and dt == F32:
        pytest.skip("two 16-bit terms")
    f = getattr(_lib(), "_ZN6kraken19launch_gemm_plannedERKNS_8GemmDescERKNS_8GemmPlanEP12ihipStream_t")
    f.restype = I
    S = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16}[dt]
    out = torch.float32 if epi in (RES, PART) else S
    # rounding of the stored type (half a unit, and twice that for ties of fp32 sums); fp32
    # sums of K products of unit-variance operands: far below 1e-5 of the result's norm
    tol = {torch.float32: 1e-5, torch.float16: 4e-4, torch.bfloat16: 3.2e-3}[out]
    if epi == HILO:
        tol = {BF16: 2e-5, F16: 1e-6}[dt]     # (2^-8)^2, and (2^-11)^2 with fp32 sums
    plans = [(TILE256, 0), (TILE128, 0)] + [(MID, nb) for nb in range(1, 7)]
    if dt != F32:
        plans.append((TILE128, 2))            # 128 x 64
    for M, N, K, batch, splits in SHAPES:
        if epi == HILO and N % 4:
            N += 4 - N % 4
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        A = torch.randn((batch, M, K), generator=g, device="cuda").to(S)
        B = (torch.randn((batch, N, K), generator=g, device="cuda") / math.sqrt(K)).to(S)
        bias = torch.randn((batch, M if epi == BIAS_M else N), generator=g, device="cuda")
        R = torch.randn((batch, M, N), generator=g, device="cuda")
        ref = torch.stack([a @ b.T for a, b in zip(A.double(), B.double())])
        if epi != PART:
            ref = ref + (bias.double()[:, :, None] if epi == BIAS_M else bias.double()[:, None])
        if epi == GELU:
            ref = torch.nn.functional.gelu(ref)
        if epi in (RES, HILO):
            ref = ref + R.double()
        planes = splits if epi == PART else 2 if epi == HILO else 1
        d = Desc(dt, epi, A.data_ptr(), B.data_ptr(), 0, bias.data_ptr(), R.data_ptr(), M, N, K,
                 K, K, N, M * K, N * K, M * N, M * N, bias.shape[1], batch, 1, 0, 0, 1,
                 splits if epi == PART else 1, batch * M * N, 0, None, None)
        for kind, nb in plans:
            C = torch.full((planes, batch, M, N), float("nan"), dtype=out, device="cuda")
            d.C = C.data_ptr()
            rc = f(ctypes.byref(d), ctypes.byref(Plan(kind, nb, d.splits)),
                   P(torch.cuda.current_stream().cuda_stream or None))
            assert rc == 0
            torch.cuda.synchronize()
            err = float((C.double().sum(0) - ref).norm() / ref.norm())
            assert err <= tol, (M, N, K, batch, splits, kind, nb, err)


# a few rows: one to four blocks of 16, column counts that are no multiple of 16 or 32, steps of
# the reduction that do not divide over the waves (some waves have none)
FEW_ROWS = [(1, 300, 64, 2), (5, 1000, 2048, 3), (16, 64, 8192, 1), (17, 33, 320, 2),
            (32, 260, 2112, 2), (33, 520, 2112, 2), (64, 130, 704, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("dual", [False, True])
@pytest.mark.parametrize("epi", [BIAS_N, GELU, RES, HILO, PART])
@pytest.mark.parametrize("dt", [F32, BF16, F16])
def test_every_few_row_plan(dt, epi, dual):
    if dt == F32 and (epi == HILO or dual) or dual and epi not in (RES, PART):
        pytest.skip("not a kernel")
    f = getattr(_lib(), "_ZN6kraken19launch_gemm_plannedERKNS_8GemmDescERKNS_8GemmPlanEP12ihipStream_t")
    f.restype = I
    S = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16}[dt]
    out = torch.float32 if epi in (RES, PART) else S
    # as above
    tol = {torch.float32: 1e-5, torch.float16: 4e-4, torch.bfloat16: 3.2e-3}[out]
    if epi == HILO:
        tol = {BF16: 2e-5, F16: 1e-6}[dt]
    for M, N, K, batch in FEW_ROWS:
        if epi == PART and K < 256:        # fewer slices than splits are refused
            continue
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        # two terms of A: the second one is the kernel's only where it reads two
        A = torch.randn((2, batch, M, K), generator=g, device="cuda").to(S)
        B = (torch.randn((batch, N, K), generator=g, device="cuda") / math.sqrt(K)).to(S)
        bias = torch.randn((batch, N), generator=g, device="cuda")
        R = torch.randn((batch, M, N), generator=g, device="cuda")
        a64 = A.double().sum(0) if dual else A[0].double()
        ref = torch.stack([a @ b.T for a, b in zip(a64, B.double())])
        if epi != PART:
            ref = ref + bias.double()[:, None]
        planes = 3 if epi == PART else 2 if epi == HILO else 1
        if epi == GELU:
            ref = torch.nn.functional.gelu(ref)
        if epi in (RES, HILO):
            ref = ref + R.double()
        d = Desc(dt, epi, A.data_ptr(), B.data_ptr(), 0, bias.data_ptr(), R.data_ptr(), M, N, K,
                 K, K, N, M * K, N * K, M * N, M * N, N, batch, 1, 0, 0, 1, 3 if epi == PART else 1, batch * M * N,
                 batch * M * K if dual else 0, None, None)
        for tw, waves in [(t, w) for t in (1, 2) for w in (4, 8, 16)]:
            C = torch.full((planes, batch, M, N), float("nan"), dtype=out, device="cuda")
            d.C = C.data_ptr()
            rc = f(ctypes.byref(d), ctypes.byref(Plan(SKINNY, tw, d.splits, waves)),
                   P(torch.cuda.current_stream().cuda_stream or None))
            if (tw, waves) not in few_row_forms(dt, M):
                assert rc != 0                # (refused by the host: not built)
                continue
            assert rc == 0
            torch.cuda.synchronize()
            err = float((C.double().sum(0) - ref).norm() / ref.norm())
            assert err <= tol, (M, N, K, batch, tw, waves, err)

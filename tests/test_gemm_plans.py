"""GEMM plans: the planner's rules (host) and every kernel, tile and epilogue a plan can name,
forced at the edges of its tiles (GPU, against fp64 products of the same operands)."""

import ctypes
import math
import os
import random
import re

import pytest
import torch

F32, BF16, F16 = 0, 1, 2
BIAS_N, GELU, RES, BIAS_M, HILO, PART, QKV = range(7)
TILE256, TILE128, MID, SKINNY = range(4)
P, I, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64


class Desc(ctypes.Structure):       # kraken::GemmDesc
    _fields_ = [("dt", I), ("epi", I), ("A", P), ("B", P), ("C", P), ("bias", P), ("R", P),
                ("M", I), ("N", I), ("K", I), ("lda", I), ("ldb", I), ("ldc", I), ("sA", L),
                ("sB", L), ("sC", L), ("sR", L), ("sBias", L), ("batch", I), ("kgroups", I),
                ("gA", L), ("gB", L), ("gBmod", I), ("splits", I), ("sPlane", L),
                ("gA2", L), ("qkv", P), ("ovf", P)]


class Qkv(ctypes.Structure):        # kraken::QkvOut
    _fields_ = [("vt", P), ("svt", L), ("cache", P), ("ldv", I), ("dq", I), ("dkv", I), ("hd", I),
                ("Hkv", I), ("max_seqs", I), ("cap", I), ("lens", I * 256)]


class Plan(ctypes.Structure):       # kraken::GemmPlan
    _fields_ = [("kind", I), ("nb", I), ("splits", I), ("waves", I)]


def _lib():
    from paper_2408_07802_amd import kraken
    return kraken.lib()


def plan(dt, epi, M, N, K, kgroups, batch, part, own_sum=False, terms=1):
    f = getattr(_lib(), "_ZN6kraken9plan_gemmENS_5DTypeEiiiiiiilb")
    f.argtypes, f.restype = [I] * 8 + [L, ctypes.c_bool], Plan
    return f(dt, epi, M, N, K, kgroups, terms, batch, part, own_sum)


@pytest.mark.parametrize("name,mirror", [("GemmDesc", Desc), ("QkvOut", Qkv), ("GemmPlan", Plan)])
def test_structs_mirror_the_header(name, mirror):
    import paper_2408_07802_amd as pkg
    with open(os.path.join(os.path.dirname(pkg.__file__), "csrc", "kraken_internal.hpp")) as f:
        body = re.search(r"struct %s \{(.*?)\n\};" % name, f.read(), re.S).group(1)
    fields = []
    for decl in re.sub(r"//.*", "", body).replace("\n", " ").split(";"):
        if not decl.strip():
            continue
        words = re.match(r"\s*((?:const )?\w+)\s*(.*)", decl)
        for item in words.group(2).split(","):
            word = re.match(r"\s*(\**)\s*(\w+)\s*(?:\[(\d+)\])?\s*$", item)
            pointer = "*" in words.group(2)
            t = P if pointer else L if words.group(1) == "int64_t" else I
            fields.append((word.group(2), t * int(word.group(3)) if word.group(3) else t))
    assert [n for n, _ in fields] == [n for n, _ in mirror._fields_]
    assert [ctypes.sizeof(t) for _, t in fields] == [ctypes.sizeof(t) for _, t in mirror._fields_]


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


# ------------------------------------------------------------------ every kernel, forced (GPU)
#
# Operands and results are laid out as a model's: K groups of A one block of rows after the
# other, K groups of B side by side in a row and used in turn (gBmod of them), results with row
# strides above N.  Everything around the results holds MARK and must keep it.

TORCH = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16}
UNIT = {torch.float32: 0.0, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}
MARK = -768.0                 # exact in every type


def launch(d, kind, nb, waves=0):
    f = getattr(_lib(), "_ZN6kraken19launch_gemm_plannedERKNS_8GemmDescERKNS_8GemmPlanEP12ihipStream_t")
    f.restype = I
    rc = f(ctypes.byref(d), ctypes.byref(Plan(kind, nb, d.splits, waves)),
           P(torch.cuda.current_stream().cuda_stream or None))
    torch.cuda.synchronize()
    return rc


def check(got, ref, unit, k, sums, what):
    """Every element within its bound: half a unit of the stored type (unit; two terms of a 16-bit
    type: that of both, and the smallest step of the second), and the rounding of fp32 sums of k
    products.  A partial sum is of the size of sums, each addition rounds it by up to 2^-24, and the
    roundings are independent: sqrt(k) of them in the mean, 32 times that for the largest of 10^6
    elements and partial sums above that size.  The norm is held to the same without the 32."""
    err = (got.double() - ref).abs()
    add = math.sqrt(k) * 2.0 ** -24 * float(sums.pow(2).mean().sqrt())
    bound = unit * ref.abs() + 32 * add + 2.0 ** -24
    assert bool((err <= bound).all()), (what, float((err / bound).max()))
    assert float(err.pow(2).mean().sqrt()) <= \
        0.75 * unit * float(ref.pow(2).mean().sqrt()) + 4 * add + 2.0 ** -24, what


class Product:
    """One GEMM: operands, its fp64 result, and a descriptor without C."""

    def __init__(self, dt, epi, M, N, K, batch, groups=1, gmod=1, pad=4, dual=False, scale=1.0):
        self.dt, self.epi, self.M, self.N, self.batch, self.groups = dt, epi, M, N, batch, groups
        S = TORCH[dt]
        g = torch.Generator(device="cuda").manual_seed(M + N + K + groups)

        def rand(*shape):
            return torch.randn(shape, generator=g, device="cuda")

        terms = 2 if dual else 1
        self.A = rand(terms, groups, batch, M, K).to(S)
        self.B = (rand(batch, N, gmod, K) / math.sqrt(K * groups * terms)).to(S)
        self.bias = rand(batch, M if epi == BIAS_M else N)
        self.ldc, self.rows = N + pad, M + 1
        self.R = rand(batch, self.rows, self.ldc)
        a64 = self.A.double().sum(0) if dual else self.A[0].double()
        b64 = self.B.double()
        self.sums = torch.stack([sum(a64[t, z] @ b64[z, :, t % gmod].T for t in range(groups))
                                 for z in range(batch)])
        ref = self.sums
        if epi != PART:
            ref = ref + (self.bias.double()[:, :, None] if epi == BIAS_M
                         else self.bias.double()[:, None])
        if epi == GELU:
            ref = torch.nn.functional.gelu(ref)
        if epi in (RES, HILO):
            ref = ref + self.R[:, :M, :N].double()
        self.ref, self.k = ref, K * groups * terms
        self.out = torch.float32 if epi in (RES, PART) else S
        size = self.rows * self.ldc
        self.d = Desc(dt, epi, self.A.data_ptr(), self.B.data_ptr(), 0, self.bias.data_ptr(),
                      self.R.data_ptr(), M, N, K, K, gmod * K, self.ldc, M * K, N * gmod * K, size,
                      size, self.bias.shape[1], batch, groups, batch * M * K, K, gmod, 1,
                      batch * size, groups * batch * M * K if dual else 0, None, None)

    def run(self, kind, nb, waves=0, splits=1, what=None):
        planes = splits if self.epi == PART else 2 if self.epi == HILO else 1
        C = torch.full((planes, self.batch, self.rows, self.ldc), MARK, dtype=self.out, device="cuda")
        self.d.C, self.d.splits = C.data_ptr(), splits
        rc = launch(self.d, kind, nb, waves)
        if rc != 0:
            return rc
        what = (self.M, self.N, self.groups, splits, kind, nb, waves, what)
        assert bool((C[:, :, self.M:] == MARK).all()) and bool((C[..., self.N:] == MARK).all()), what
        unit = UNIT[self.out] ** (2 if self.epi == HILO else 1)
        check(C[:, :, :self.M, :self.N].double().sum(0), self.ref, unit, self.k, self.sums, what)
        return 0


# (M, N, K, batch, K splits): one row past and short of tiles of 128 and 256, column counts
# that are no multiple of a tile or of 4, splits of unequal length, a single slice
SHAPES = [(65, 96, 64, 1, 1), (127, 130, 192, 2, 3), (128, 160, 128, 1, 2), (129, 257, 320, 2, 5),
          (255, 64, 640, 1, 4), (257, 320, 512, 2, 8), (300, 33, 448, 3, 2)]


def all_plans(dt):
    plans = [(TILE256, 0), (TILE128, 0)] + [(MID, nb) for nb in range(1, 7)]
    return plans + ([(TILE128, 2)] if dt != F32 else [])      # 128 x 64


@pytest.mark.gpu
@pytest.mark.parametrize("epi", [BIAS_N, GELU, RES, BIAS_M, HILO, PART])
@pytest.mark.parametrize("dt", [F32, BF16, F16])
def test_every_plan_at_tile_edges(dt, epi):
    if epi == HILO and dt == F32:
        pytest.skip("two 16-bit terms")
    for M, N, K, batch, splits in SHAPES:
        if epi == HILO and N % 4:
            N += 4 - N % 4
        for pad in (4, 3):                    # rows that whole groups of 4 can and cannot be stored to
            if epi == HILO and pad == 3:
                continue
            p = Product(dt, epi, M, N, K, batch, pad=pad)
            for kind, nb in all_plans(dt):
                assert p.run(kind, nb, splits=splits if epi == PART else 1, what=pad) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("groups,gmod", [(3, 3), (6, 3), (4, 1)])
@pytest.mark.parametrize("epi", [RES, PART])
@pytest.mark.parametrize("dt", [F32, BF16, F16])
def test_k_groups_and_splits_that_begin_inside_them(dt, epi, groups, gmod):
    """W_concat's reduction: groups of K, the weights of gmod groups used in turn (two terms: twice
    each).  Splits of 2, 5 and 7 begin inside groups, at their borders and across the wrap."""
    for M, N, K, batch in ((65, 100, 192, 1), (130, 68, 128, 2), (257, 132, 64, 1)):
        p = Product(dt, epi, M, N, K, batch, groups, gmod)
        for kind, nb in all_plans(dt):
            for splits in (2, 5, 7) if epi == PART else (1,):
                if splits <= K // (32 if dt == F32 else 64) * groups:
                    assert p.run(kind, nb, splits=splits) == 0


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
    for M, N, K, batch in FEW_ROWS:
        for groups, splits in ((1, 3), (3, 5)):
            if epi == PART and K // (32 if dt == F32 else 64) * groups < splits:
                continue                      # fewer slices than splits are refused
            if groups * K > 7000 or groups > 1 and epi not in (RES, PART):
                continue
            p = Product(dt, epi, M, N, K, batch, groups, groups, dual=dual)
            for tw, waves in [(t, w) for t in (1, 2) for w in (4, 8, 16)]:
                rc = p.run(SKINNY, tw, waves, splits if epi == PART else 1)
                # (a form that is not built is refused by the host)
                assert (rc == 0) == ((tw, waves) in few_row_forms(dt, M)), (M, tw, waves)


# (heads, key/value heads, head size): borders of Q, K and V inside and on the tiles of every
# kernel; 416 and 320 columns are no multiple of 32 nb for some nb
QKV_HEADS = [(3, 2, 32), (4, 4, 32), (3, 1, 64), (5, 2, 64), (2, 1, 128), (4, 2, 128)]


def qkv_plans(dt, M):
    return [(MID, nb, 0) for nb in range(1, 7)] + [(SKINNY, t, w) for t, w in few_row_forms(dt, M)]


@pytest.mark.gpu
@pytest.mark.parametrize("decode", [False, True])
@pytest.mark.parametrize("dt", [F32, BF16, F16])
def test_qkv_columns_go_to_their_places(dt, decode):
    """The merged projection: Q | K rows and V transposed (prefill), or Q rows and K and V at each
    sequence's place in the cache (decode step), and nothing anywhere else."""
    S, batch, K = TORCH[dt], 2, 192
    rng = random.Random(3)
    for M in (1, 7, 16, 29, 64, 70, 128, 133, 256) + (() if decode else (300,)):
        for H, Hkv, hd in QKV_HEADS:
            dq, dkv = H * hd, Hkv * hd
            N = dq + 2 * dkv
            p = Product(dt, BIAS_N, M, N, K, batch, pad=0)
            d, cap, max_seqs = p.d, 9, M + 2
            lens = [rng.randint(0, cap - 1) for _ in range(M)]
            ldv = (M + 63) // 64 * 64
            cols = dq if decode else dq + dkv
            d.epi, d.ldc, d.sC = QKV, cols + 4, (M + 1) * (cols + 4)
            for kind, nb, waves in qkv_plans(dt, M):
                C = torch.full((batch, M + 1, cols + 4), MARK, dtype=S, device="cuda")
                vt = torch.full((batch, dkv, ldv), MARK, dtype=S, device="cuda")
                cache = torch.full((batch, 2, max_seqs, Hkv, cap, hd), MARK, dtype=S, device="cuda")
                q = Qkv(vt.data_ptr(), dkv * ldv, cache.data_ptr() if decode else None, ldv, dq, dkv,
                        hd, Hkv, max_seqs, cap)
                for b, n in enumerate(lens):
                    if decode:
                        q.lens[b] = n
                d.C, d.qkv, d.splits = C.data_ptr(), ctypes.addressof(q), 1
                assert launch(d, kind, nb, waves) == 0
                what = (M, H, Hkv, hd, kind, nb, waves)
                got = torch.empty((batch, M, N), dtype=S, device="cuda")
                got[..., :cols] = C[:, :M, :cols]
                assert bool((C[:, M:] == MARK).all()) and bool((C[..., cols:] == MARK).all()), what
                if decode:
                    slot = torch.arange(M, device="cuda")
                    at = torch.tensor(lens, device="cuda")
                    rows = cache[:, :, slot, :, at]                  # [M][batch][2][Hkv][hd]
                    got[..., dq:] = rows.permute(1, 0, 2, 3, 4).reshape(batch, M, 2 * dkv)
                    cache[:, :, slot, :, at] = MARK
                    assert bool((vt == MARK).all()), what
                else:
                    got[..., cols:] = vt[:, :, :M].transpose(1, 2)
                    assert bool((vt[:, :, M:] == MARK).all()), what
                assert bool((cache == MARK).all()), what
                check(got, p.ref, UNIT[S], p.k, p.sums, what)

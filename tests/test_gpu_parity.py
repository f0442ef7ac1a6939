"""GPU parity: every entry point of the C ABI against the fp64 CPU oracle,
element by element, on the same seeded inputs.

Bars (stated by the benchmark spec): Philox words bit-exact; floating
outputs within relative Frobenius error 1e-5 on the fp32 matrix-core path
(ranks 8/16/32) and 2e-2 on the bf16 matrix-core path (ranks 64/128/256).
"""
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
from paper_2402_03293_amd import flora, workloads  # noqa: E402

pytestmark = pytest.mark.gpu

from parity_bars import TOL_BF16, TOL_F32, tol_for, update_bar  # noqa: E402
DEV = "cuda:0"




def to64(t):
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def rel_fro(x, ref):
    ref = np.asarray(ref, dtype=np.float64)
    x = np.asarray(x, dtype=np.float64)
    den = np.linalg.norm(ref)
    return np.linalg.norm(x - ref) / (den if den > 0 else 1.0)


def rand(shape, seed, dtype=torch.float32, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (scale * torch.randn(*shape, generator=g)).to(dtype).to(DEV).contiguous()


def sync():
    torch.cuda.synchronize()


# ------------------------------------------------------------- generator
@pytest.mark.parametrize("m,r", [(300, 32), (64, 8), (1025, 256), (7, 4)])
def test_philox_words_bit_exact_and_normals_close(m, r):
    seed = 0xDEADBEEF12345678
    nq = r // 4
    raw = torch.empty((m, nq, 4), dtype=torch.int32, device=DEV)
    A = torch.empty((m, r), dtype=torch.float32, device=DEV)
    flora.debug_generate(seed, m, r, A, raw)
    sync()
    got = raw.cpu().numpy().view(np.uint32)
    mm = min(m, 200)
    want = oracle.raw_words_matrix(seed, mm, r)
    assert np.array_equal(got[:mm], want)
    Aref = oracle.materialise_A(seed, m, r)
    Ag = to64(A)
    err = np.abs(Ag - Aref).max() * math.sqrt(r)
    assert err < 2e-5, err                      # per-entry error of a standard normal
    assert rel_fro(Ag, Aref) < 2e-6


def test_generator_error_statistics_large_sample():
    # 2^20 normals: RMS error of the hardware log2 / sin / cos path against fp64
    seed, m, r = 77, 4096, 256
    A = torch.empty((m, r), dtype=torch.float32, device=DEV)
    flora.debug_generate(seed, m, r, A, None)
    sync()
    Aref = oracle.materialise_A(seed, m, r)
    Ag = to64(A)
    rel = rel_fro(Ag, Aref)
    mx = np.abs(Ag - Aref).max() * math.sqrt(r)
    print("generator: rel fro %.3e  max abs (sigma units) %.3e" % (rel, mx))
    assert rel < 2e-6
    assert mx < 5e-5


def test_derive_seed_matches_oracle():
    for g, l, e in [(0, 0, 0), (5, 3, 9), (2 ** 63 + 11, 383, 2 ** 33 + 5)]:
        assert flora.derive_seed(g, l, e) == oracle.derive_seed(g, l, e)


# -------------------------------------------------------------- compress
F32_CASES = [
    # n, m, r
    (256, 256, 8), (130, 200, 16), (77, 70, 32), (5, 7, 8), (64, 64, 16), (1, 1, 8),
    (200, 1000, 16), (65, 129, 32),
]
BF16_CASES = [(300, 520, 64), (64, 40, 64), (100, 1003, 128), (257, 264, 256), (33, 96, 256), (1, 8, 64)]


@pytest.mark.parametrize("n,m,r", F32_CASES)
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_compress_fp32_path(n, m, r, gdt):
    seed = 1000 + n + m + r
    G = rand((n, m), seed, torch.float32 if gdt == "f32" else torch.bfloat16)
    S0 = rand((n, r), seed + 1)
    st = S0.clone()
    mats = flora.matrices([(n, m)], grads=[G], states=[st], seeds=[seed])
    a, b = 0.9, 0.1
    flora.compress(mats, r, flora.F32 if gdt == "f32" else flora.BF16, a, b)
    sync()
    ref = oracle.compress(to64(G), r, seed, state=to64(S0), a=a, b=b)
    assert rel_fro(to64(st), ref) < TOL_F32
    # a = 0 overwrites whatever the state held (NaN included)
    st2 = torch.full((n, r), float("nan"), device=DEV)
    mats2 = flora.matrices([(n, m)], grads=[G], states=[st2], seeds=[seed])
    flora.compress(mats2, r, flora.F32 if gdt == "f32" else flora.BF16, 0.0, 1.0)
    sync()
    assert rel_fro(to64(st2), oracle.compress(to64(G), r, seed)) < TOL_F32


@pytest.mark.parametrize("n,m,r", BF16_CASES)
def test_compress_bf16_path(n, m, r):
    seed = 2000 + n + m + r
    G = rand((n, m), seed, torch.bfloat16)
    S0 = rand((n, r), seed + 1)
    st = S0.clone()
    mats = flora.matrices([(n, m)], grads=[G], states=[st], seeds=[seed])
    flora.compress(mats, r, flora.BF16, 0.9, 0.1)
    sync()
    # compare the G A part alone too: the carried-over state would mask its error
    st2 = torch.zeros((n, r), device=DEV)
    mats2 = flora.matrices([(n, m)], grads=[G], states=[st2], seeds=[seed])
    flora.compress(mats2, r, flora.BF16, 1.0, 1.0)
    sync()
    ref = oracle.compress(to64(G), r, seed, state=to64(S0), a=0.9, b=0.1)
    ref2 = oracle.compress(to64(G), r, seed)
    assert rel_fro(to64(st), ref) < TOL_BF16
    e = rel_fro(to64(st2), ref2)
    assert e < TOL_BF16, e
    assert e < 6e-3          # one bf16-rounded operand: about 2^-9 / sqrt(3)


# fp32 gradients at the bf16-path ranks: rounded to bf16 in registers, same bar as bf16 gradients
@pytest.mark.parametrize("mt", [0, 1, 2, 4])
@pytest.mark.parametrize("n,m,r", [(300, 520, 64), (257, 1001, 128), (1100, 264, 256), (70, 36, 256), (513, 31, 64)])
def test_compress_bf16_path_fp32_gradients(n, m, r, mt):
    seed = 2500 + n + m + r
    G = rand((n, m), seed)
    S0 = rand((n, r), seed + 1)
    st = S0.clone()
    st2 = torch.zeros((n, r), device=DEV)
    flora.set_tuning("compress_bf16_mt", mt)
    try:
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[st], seeds=[seed]), r, flora.F32, 0.9, 0.1)
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[st2], seeds=[seed]), r, flora.F32, 1.0, 1.0)
        sync()
    finally:
        flora.set_tuning("compress_bf16_mt", 0)
    assert rel_fro(to64(st), oracle.compress(to64(G), r, seed, state=to64(S0), a=0.9, b=0.1)) < TOL_BF16
    e = rel_fro(to64(st2), oracle.compress(to64(G), r, seed))
    assert e < TOL_BF16 and e < 8e-3, e          # two bf16-rounded operands
    # rounding G first and multiplying exactly is what the kernel does: against that it is tight
    Gb = to64(G.to(torch.bfloat16))
    assert rel_fro(to64(st2), oracle.compress(Gb, r, seed)) < 6e-3


# every launch shape of the bf16 compress kernel, forced through the tuning hook: the narrow
# kernel (128 / 256 / 512 rows per workgroup) and the wide one (8 / 16 / 32: 512 / 256 / 128 rows, rank
# slices of 128),
# on shapes with ragged row blocks, a ragged last column tile and odd / even tile counts
@pytest.mark.parametrize("mt", [1, 2, 4, 8, 16, 32])
@pytest.mark.parametrize("n,m,r", [(700, 520, 256), (1100, 64, 128), (97, 1160, 64), (513, 200, 256)])
def test_compress_bf16_every_launch_shape(n, m, r, mt):
    seed = 2500 + n + m + r
    G = rand((n, m), seed, torch.bfloat16)
    S0 = rand((n, r), seed + 1)
    st = S0.clone()
    st2 = torch.zeros((n, r), device=DEV)
    flora.set_tuning("compress_bf16_mt", mt)
    try:
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[st], seeds=[seed]), r, flora.BF16, 0.9, 0.1)
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[st2], seeds=[seed]), r, flora.BF16, 1.0, 1.0)
        sync()
    finally:
        flora.set_tuning("compress_bf16_mt", 0)
    ref = oracle.compress(to64(G), r, seed, state=to64(S0), a=0.9, b=0.1)
    ref2 = oracle.compress(to64(G), r, seed)
    assert rel_fro(to64(st), ref) < TOL_BF16
    e = rel_fro(to64(st2), ref2)
    assert e < 6e-3, e
    # row by row as well: a wrong row block would hide in the Frobenius norm of a large matrix
    rows = np.linalg.norm(to64(st2) - ref2, axis=1) / np.linalg.norm(ref2, axis=1)
    assert rows.max() < TOL_BF16, (int(rows.argmax()), float(rows.max()))


# the fp32 kernel with the pieces and column groups it chooses: a launch of few workgroups (pieces of 256
# columns, two column groups), one of more (512), and sets large enough for 1024.  Products and
# sums are fp32: about sqrt(m) 2^-24 = 3e-6 at the widest, TOL_F32 as for the other shapes.
@pytest.mark.parametrize("count,n,m", [(1, 33, 1), (1, 70, 257), (2, 65, 515), (130, 64, 1027), (620, 63, 1030), (1300, 31, 2053)])
@pytest.mark.parametrize("r", [8, 32])
def test_compress_f32_pieces(r, count, n, m):
    G = rand((count, n, m + 4 - m % 4), 2500 + n + m, torch.float32)
    Gs = [G[l].view(-1)[:n * m].view(n, m) for l in range(count)]
    states = [torch.zeros((n, r), device=DEV) for _ in range(count)]
    seeds = [2500 + l for l in range(count)]
    mats = flora.matrices([(n, m)] * count, grads=Gs, states=states, seeds=seeds)
    for _ in range(2):                            # (the arrival counters must be back at zero)
        flora.compress(mats, r, flora.F32, 0.0, 1.0)
        sync()
        for l in sorted({0, count // 2, count - 1}):
            assert rel_fro(to64(states[l]), oracle.compress(to64(Gs[l]), r, seeds[l])) < TOL_F32


# matrices of one tile of columns: the round after it multiplies zeros, and whatever the other LDS buffer holds must
# not turn them into NaN (a decompression of NaNs leaves its operands in every compute unit's LDS)
@pytest.mark.parametrize("gdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,m,r", [(130, 64, 8), (130, 40, 16), (70, 64, 32), (65, 64, 16)])
def test_compress_f32_one_tile_after_nans(n, m, r, gdt):
    S, big = torch.full((4096, 256), float("nan"), device=DEV), torch.empty(4096, 4096, device=DEV)
    G, C = rand((n, m), 77).to(gdt).contiguous(), torch.zeros(n, r, device=DEV)
    for _ in range(3):
        flora.decompress(flora.matrices([(4096, 4096)], states=[S], seeds=[1]), 256, 1.0, [big], flora.F32)
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[C], seeds=[3]), r, flora.F32 if gdt == torch.float32 else flora.BF16, 0.0, 1.0)
        sync()
        assert rel_fro(to64(C), oracle.compress(to64(G), r, 3)) < TOL_F32


# rows of G that start anywhere (odd widths, widths that are no multiple of 8, fp32 gradients) in the
# wide kernel: widths around a tile of 64 columns and around the pieces of a load, row counts around a
# wave's and a workgroup's, whole rows and shared columns.  The matrix lies between NaNs: whatever a
# load fetches beside its row must not reach the result.  Bar: one rounded operand (A; with fp32
# gradients G is compared as the kernel rounds it), about 2^-9 / sqrt(3) = 1.1e-3 on a large matrix;
# the smallest have a handful of terms per entry, hence 6e-3 as for the other launch shapes.
@pytest.mark.parametrize("combine", [1, 2])       # shared columns added by the last part to arrive, or by a launch
@pytest.mark.parametrize("mt,kc", [(8, 0), (16, 64), (32, 0), (32, 192)])
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
@pytest.mark.parametrize("n,m,r", [(33, 1, 64), (130, 7, 128), (257, 63, 256), (97, 65, 64), (513, 127, 128), (31, 66, 256),
                                   (300, 130, 64), (129, 333, 256), (1030, 961, 64), (64, 1283, 128)])
def test_compress_bf16_rows_that_start_anywhere(n, m, r, gdt, mt, kc, combine):
    seed = 2600 + n + m + r
    dt = torch.float32 if gdt == "f32" else torch.bfloat16
    buf = torch.full((n * m + 128,), float("nan"), device=DEV, dtype=dt)
    G = buf[64:64 + n * m].view(n, m)
    G.copy_(rand((n, m), seed, dt))
    st = torch.zeros((n, r), device=DEV)
    mats = flora.matrices([(n, m)], grads=[G], states=[st], seeds=[seed])
    ref = oracle.compress(to64(G.to(torch.bfloat16)), r, seed)
    flora.set_tuning("compress_bf16_mt", mt)
    flora.set_tuning("compress_splitk_cols", kc)
    flora.set_tuning("compress_combine", combine)
    try:
        for step in range(2):                     # (the arrival counters must be back at zero)
            flora.compress(mats, r, flora.F32 if gdt == "f32" else flora.BF16, 0.0, 1.0)
            sync()
            assert rel_fro(to64(st), ref) < 6e-3
            rows = np.linalg.norm(to64(st) - ref, axis=1) / np.linalg.norm(ref, axis=1)
            assert rows.max() < TOL_BF16, (int(rows.argmax()), float(rows.max()))
    finally:
        flora.set_tuning("compress_bf16_mt", 0)
        flora.set_tuning("compress_splitk_cols", 0)
        flora.set_tuning("compress_combine", 0)


# Shared columns added to an old state (a != 0), by the last part to arrive and by a launch of their own: aligned
# and odd rows, row blocks that are not full, parts that differ in number between the matrices.
@pytest.mark.parametrize("combine", [1, 2])
@pytest.mark.parametrize("r,mt,kc", [(64, 32, 128), (128, 16, 192), (256, 8, 384)])
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
def test_compress_shared_columns_with_an_old_state(r, mt, kc, gdt, combine):
    dt = torch.float32 if gdt == "f32" else torch.bfloat16
    for shapes in ([(300, 1160), (70, 200), (129, 64)], [(300, 1161), (70, 199), (513, 1030)]):
        G = [rand(s, 2700 + r + l, dt) for l, s in enumerate(shapes)]
        st = [rand((n, r), 2800 + l) for l, (n, _) in enumerate(shapes)]
        ref = [oracle.compress(to64(G[l].to(torch.bfloat16)), r, 60 + l, state=to64(st[l]), a=0.9, b=0.1) for l in range(len(shapes))]
        mats = flora.matrices(shapes, grads=G, states=st, seeds=[60 + l for l in range(len(shapes))])
        flora.set_tuning("compress_bf16_mt", mt)
        flora.set_tuning("compress_splitk_cols", kc)
        flora.set_tuning("compress_combine", combine)
        try:
            flora.compress(mats, r, flora.F32 if gdt == "f32" else flora.BF16, 0.9, 0.1)
            sync()
        finally:
            flora.set_tuning("compress_bf16_mt", 0)
            flora.set_tuning("compress_splitk_cols", 0)
            flora.set_tuning("compress_combine", 0)
        for l in range(len(shapes)):
            assert rel_fro(to64(st[l]), ref[l]) < 6e-3, shapes[l]


# the wide kernel with the columns of a row block shared between workgroups (partial products
# combined by the last workgroup to arrive): several parts, ragged last part, two launches in a
# row on the same descriptor set (the arrival counters must be back at zero), grouped matrices
@pytest.mark.parametrize("mt", [8, 16, 32])
@pytest.mark.parametrize("kc", [64, 192, 448])
@pytest.mark.parametrize("r", [64, 256])
def test_compress_bf16_shared_columns(r, kc, mt):
    shapes = [(300, 520), (520, 1160), (64, 64), (257, 200)]
    seeds = [2700 + r + l for l in range(len(shapes))]
    Gs = [[rand(s, 2800 + 10 * step + l, torch.bfloat16) for l, s in enumerate(shapes)] for step in range(2)]
    states = [torch.zeros((n, r), device=DEV) for n, _ in shapes]
    flora.set_tuning("compress_bf16_mt", mt)
    flora.set_tuning("compress_splitk_cols", kc)
    try:
        mats = flora.matrices(shapes, grads=Gs[0], states=states, seeds=seeds)
        flora.compress(mats, r, flora.BF16, 0.0, 1.0)
        first = [st.clone() for st in states]
        flora.compress(mats, r, flora.BF16, 0.5, 2.0)          # same plan, same gradients
        mats2 = flora.matrices(shapes, grads=Gs[1], states=states, seeds=seeds)
        flora.compress(mats2, r, flora.BF16, 1.0, 1.0)
        sync()
    finally:
        flora.set_tuning("compress_bf16_mt", 0)
        flora.set_tuning("compress_splitk_cols", 0)
    for l, (n, m) in enumerate(shapes):
        ref1 = oracle.compress(to64(Gs[0][l]), r, seeds[l])
        e1 = rel_fro(to64(first[l]), ref1)
        assert e1 < 6e-3, (l, e1)
        rows = np.linalg.norm(to64(first[l]) - ref1, axis=1) / np.linalg.norm(ref1, axis=1)
        assert rows.max() < TOL_BF16, (l, int(rows.argmax()), float(rows.max()))
        ref = oracle.compress(to64(Gs[1][l]), r, seeds[l], state=2.5 * ref1)
        assert rel_fro(to64(states[l]), ref) < 6e-3


# compressed EMA of the second moment: the square is taken in registers on the way in.  Every
# rank, both gradient types, ragged shapes and unaligned rows, forced launch shapes, two steps of
# the EMA; then the state decompresses to what the oracle's state decompresses to.
@pytest.mark.parametrize("gdt", ["f32", "bf16"])
@pytest.mark.parametrize("n,m,r,mt", [(70, 200, 8, 0), (130, 1001, 16, 2), (257, 520, 32, 0), (300, 520, 64, 0),
                                      (257, 1001, 128, 2), (700, 264, 256, 4), (513, 31, 64, 1),
                                      (700, 264, 256, 8), (1100, 520, 128, 16), (530, 1160, 64, 8),
                                      # rows that start anywhere (odd widths, even ones off 16 bytes) in the wide kernel
                                      (257, 1001, 128, 16), (530, 333, 64, 8), (97, 1283, 256, 32), (140, 522, 64, 0),
                                      (257, 1001, 256, 0), (65, 66, 128, 0)])
def test_compress_mapped_square(n, m, r, mt, gdt):
    dt = torch.float32 if gdt == "f32" else torch.bfloat16
    fd = flora.F32 if gdt == "f32" else flora.BF16
    seed, beta2 = 4100 + n + m + r, 0.9
    G1, G2 = rand((n, m), seed, dt), rand((n, m), seed + 1, dt, scale=3.0)
    st = torch.zeros((n, r), device=DEV)
    knob = "compress_f32_mt" if r <= 32 else "compress_bf16_mt"
    flora.set_tuning(knob, mt)
    try:
        flora.compress_mapped(flora.matrices([(n, m)], grads=[G1], states=[st], seeds=[seed]), r, fd,
                              flora.INPUT_SQUARE, 0.0, 1.0 - beta2)
        flora.compress_mapped(flora.matrices([(n, m)], grads=[G2], states=[st], seeds=[seed]), r, fd,
                              flora.INPUT_SQUARE, beta2, 1.0 - beta2)
        ident = torch.zeros((n, r), device=DEV)
        flora.compress_mapped(flora.matrices([(n, m)], grads=[G1], states=[ident], seeds=[seed]), r, fd,
                              flora.INPUT_IDENTITY, 0.0, 1.0)
        plain = torch.zeros((n, r), device=DEV)
        flora.compress(flora.matrices([(n, m)], grads=[G1], states=[plain], seeds=[seed]), r, fd, 0.0, 1.0)
        sync()
    finally:
        flora.set_tuning(knob, 0)
    ref = oracle.compress_mapped(to64(G1), r, seed, "square", a=0.0, b=1.0 - beta2)
    ref = oracle.compress_mapped(to64(G2), r, seed, "square", state=ref, a=beta2, b=1.0 - beta2)
    e = rel_fro(to64(st), ref)
    assert e < (TOL_F32 if r <= 32 else 6e-3), e
    rows = np.linalg.norm(to64(st) - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert rows.max() < tol_for(r), (int(rows.argmax()), float(rows.max()))
    assert torch.equal(ident, plain)       # the identity map is flora_compress


def test_compress_mapped_grouped_and_errors():
    shapes = [(96, 160), (40, 72), (200, 64)]
    r = 16
    Gs = [rand(s, 4300 + l) for l, s in enumerate(shapes)]
    states = [torch.zeros((n, r), device=DEV) for n, _ in shapes]
    seeds = [4400 + l for l in range(len(shapes))]
    mats = flora.matrices(shapes, grads=Gs, states=states, seeds=seeds)
    flora.compress_mapped(mats, r, flora.F32, flora.INPUT_SQUARE, 0.0, 1.0)
    sync()
    for l in range(len(shapes)):
        assert rel_fro(to64(states[l]), oracle.compress_mapped(to64(Gs[l]), r, seeds[l], "square")) < TOL_F32
    with pytest.raises(flora.FloraError):
        flora.compress_mapped(mats, r, flora.F32, 2, 0.0, 1.0)
    with pytest.raises(flora.FloraError):
        flora.compress_mapped(mats, 48, flora.F32, flora.INPUT_SQUARE, 0.0, 1.0)


# the fp32 matrix-core kernel with shared columns, every rank, both gradient types, 1 / 2 / 4
# column groups per workgroup, ragged parts, two launches in a row on one descriptor set
@pytest.mark.parametrize("kg", [1, 2, 4])
@pytest.mark.parametrize("r,gdt", [(8, "f32"), (16, "f32"), (32, "bf16"), (16, "bf16")])
def test_compress_fp32_path_shared_columns(r, gdt, kg):
    shapes = [(130, 520), (64, 1160), (33, 64), (200, 203)]
    tdt = torch.float32 if gdt == "f32" else torch.bfloat16
    fdt = flora.F32 if gdt == "f32" else flora.BF16
    seeds = [2900 + r + l for l in range(len(shapes))]
    Gs = [rand(s_, 2950 + l, tdt) for l, s_ in enumerate(shapes)]
    states = [torch.full((n, r), float("nan"), device=DEV) for n, _ in shapes]
    flora.set_tuning("compress_f32_kgroups", kg)
    flora.set_tuning("compress_splitk_cols", 128)
    try:
        mats = flora.matrices(shapes, grads=Gs, states=states, seeds=seeds)
        flora.compress(mats, r, fdt, 0.0, 1.0)
        flora.compress(mats, r, fdt, 0.5, 2.0)
        sync()
    finally:
        flora.set_tuning("compress_f32_kgroups", 0)
        flora.set_tuning("compress_splitk_cols", 0)
    for l in range(len(shapes)):
        ref = 2.5 * oracle.compress(to64(Gs[l]), r, seeds[l])
        assert rel_fro(to64(states[l]), ref) < TOL_F32, l
        rows = np.linalg.norm(to64(states[l]) - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert rows.max() < TOL_F32, (l, int(rows.argmax()), float(rows.max()))


def test_compress_grouped_many_matrices_and_accumulation():
    shapes = [(96, 128), (64, 300), (130, 64), (32, 32), (200, 72)]
    r, tau = 16, 3
    seeds = [50 + l for l in range(len(shapes))]
    states = [torch.zeros((n, r), device=DEV) for n, _ in shapes]
    ref = [np.zeros((n, r)) for n, _ in shapes]
    for step in range(tau):
        Gs = [rand(s, 300 + 10 * step + l) for l, s in enumerate(shapes)]
        mats = flora.matrices(shapes, grads=Gs, states=states, seeds=seeds)
        flora.compress(mats, r, flora.F32, 1.0, 1.0)
        sync()
        for l in range(len(shapes)):
            ref[l] = oracle.compress(to64(Gs[l]), r, seeds[l], state=ref[l])
    for l in range(len(shapes)):
        assert rel_fro(to64(states[l]), ref[l]) < TOL_F32


@pytest.mark.parametrize("r,gdt,kc", [(64, "bf16", 0), (256, "bf16", 128), (16, "f32", 128), (32, "bf16", 64)])
def test_compress_is_bitwise_repeatable(r, gdt, kc):
    # also with shared columns: whichever workgroup arrives last adds the partial products in
    # the same order
    n, m = 300, 1032
    tdt = torch.float32 if gdt == "f32" else torch.bfloat16
    fdt = flora.F32 if gdt == "f32" else flora.BF16
    G = rand((n, m), 9, tdt)
    outs = []
    flora.set_tuning("compress_splitk_cols", kc)
    try:
        for _ in range(4):
            st = torch.zeros((n, r), device=DEV)
            flora.compress(flora.matrices([(n, m)], grads=[G], states=[st], seeds=[4]), r, fdt)
            sync()
            outs.append(st.cpu().numpy())
    finally:
        flora.set_tuning("compress_splitk_cols", 0)
    assert all(np.array_equal(outs[0], o) for o in outs[1:])


# ------------------------------------------------------------ decompress
@pytest.mark.parametrize("n,m,r", F32_CASES + BF16_CASES)
@pytest.mark.parametrize("odt", ["f32", "bf16"])
def test_decompress(n, m, r, odt):
    seed = 3000 + n + m + r
    S = rand((n, r), seed)
    out = torch.full((n, m), float("nan"), device=DEV,
                     dtype=torch.float32 if odt == "f32" else torch.bfloat16)
    mats = flora.matrices([(n, m)], states=[S], seeds=[seed])
    alpha = 0.125
    flora.decompress(mats, r, alpha, [out], flora.F32 if odt == "f32" else flora.BF16)
    sync()
    ref = oracle.decompress(to64(S), m, seed, alpha=alpha)
    tol = tol_for(r)
    if odt == "bf16":
        tol = max(tol, 4e-3)                     # the output itself is rounded to bf16
    assert rel_fro(to64(out), ref) < tol


# Decompression into bf16 at ranks 16 and 32 as products of bf16 parts: rows and columns around the 32 of a tile, a state
# whose rows differ by 2^80, and rows that are not finite (fp32 products then): an infinity keeps the sign of the
# entry it meets, a NaN fills its row, the largest values stay finite.  Half a bf16 step of the value, and the sum's own error.
@pytest.mark.parametrize("n,m", [(1, 1), (33, 31), (64, 129), (95, 1000)])
@pytest.mark.parametrize("r", [16, 32])
def test_decompress_into_bf16_by_parts(n, m, r):
    S = rand((n, r), 3) * torch.exp2(torch.arange(n, device=DEV) % 81 - 40.0).view(-1, 1)
    inf = float("inf")
    odd = {i: v for i, v in {5: inf, 32: float("nan"), 60: -inf, 63: 3.3e38}.items() if i < n}
    for i, v in odd.items():
        S[i, i % r] = v
    out = torch.empty((n, m), dtype=torch.bfloat16, device=DEV)
    flora.decompress(flora.matrices([(n, m)], states=[S], seeds=[8]), r, 1.0, [out], flora.BF16)
    sync()
    got = to64(out)
    A = oracle.compress(np.eye(m), r, 8)
    rows = [i for i in range(n) if i not in odd]
    ref = to64(S)[rows] @ A.T
    size = np.linalg.norm(to64(S)[rows], axis=1, keepdims=True) * np.linalg.norm(A, axis=1)[None, :]
    assert (np.abs(got[rows] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-6 * size).all()
    for i, v in odd.items():
        if np.isnan(v):
            assert np.isnan(got[i]).all()
        elif np.isinf(v):
            assert np.array_equal(got[i], np.sign(v) * np.sign(A[:, i % r]) * inf)
        else:
            fits = np.abs(v * A[:, i % r]) < 3.2e38
            assert np.abs(got[i][fits] / (v * A[fits, i % r]) - 1).max() < 1e-2


# bf16 gradients at ranks up to 32 as products of bf16 parts of A (m % 8 == 0; else the fp32 instruction): columns around
# the 64 of a tile and the pieces, one tile, shared columns, rows around the 16, 64 and 128 of a wave and a workgroup.
# Bar: fp32 sums of this length, 2^-24 sqrt(m), and the generator's share.
@pytest.mark.parametrize("n,m,count", [(1, 8, 1), (63, 56, 2), (65, 64, 1), (17, 72, 3), (130, 520, 1), (64, 1032, 5), (129, 4096, 3), (100, 68, 2), (129, 2048, 160)])
@pytest.mark.parametrize("r", [8, 16, 32])
def test_compress_bf16_parts(n, m, count, r):
    G = [rand((n, m), 40 + l).to(torch.bfloat16) for l in range(count)]
    S0 = [rand((n, r), 90 + l) for l in range(count)]
    S = [x.clone() for x in S0]
    seeds = [1000 + l for l in range(count)]
    flora.compress(flora.matrices([(n, m)] * count, grads=G, states=S, seeds=seeds), r, flora.BF16, 0.5, 2.0)
    sync()
    for l in sorted({0, count // 2, count - 1}):
        ref = oracle.compress(to64(G[l]), r, seeds[l], state=to64(S0[l]), a=0.5, b=2.0)
        assert rel_fro(to64(S[l]), ref) < 2.0 ** -24 * m ** 0.5 + 4e-7, l


# ... with 128 rows per workgroup (r = 32): shared columns, and whole rows in one column group; the last block short.
@pytest.mark.parametrize("n,m,count,kc", [(257, 2048, 80, 512), (65537, 80, 8, 0)])
def test_compress_bf16_parts_of_128_rows(n, m, count, kc):
    r = 32
    _, info = flora.debug_work_items(0, [(n, m)] * count, r, flora.BF16)
    assert (int(info[0]), int(info[2])) == (2, kc)
    G = [rand((n, m), 140 + l).to(torch.bfloat16) for l in range(count)]
    S0 = [rand((n, r), 190 + l) for l in range(count)]
    S = [x.clone() for x in S0]
    G[1][n - 1, m - 1] = float("inf")            # (its workgroup takes fp32 products)
    flora.compress(flora.matrices([(n, m)] * count, grads=G, states=S, seeds=list(range(count))), r, flora.BF16, 0.5, 2.0)
    sync()
    assert np.array_equal(to64(S[1][n - 1]), np.sign(oracle.compress(np.eye(m), r, 1)[m - 1]) * np.inf)
    G[1][n - 1] = 0
    S[1][n - 1] = 0.5 * S0[1][n - 1]
    for l in (0, 1, count - 1):
        ref = oracle.compress(to64(G[l]), r, l, state=to64(S0[l]), a=0.5, b=2.0)
        assert rel_fro(to64(S[l]), ref) < 2.0 ** -24 * m ** 0.5 + 4e-7, l


# ... infinities keep the sign of the entry of A that they meet, NaNs and opposite infinities are NaNs, other rows are those of
# the finite gradient.
@pytest.mark.parametrize("r,m", [(8, 64), (16, 1024), (32, 640)])
def test_compress_bf16_parts_of_gradients_that_are_not_finite(r, m):
    n, inf = 150, float("inf")
    G = rand((n, m), 5).to(torch.bfloat16)
    clean = G.clone()
    G[3, 5], G[70, m - 1], G[129, 0], G[149, 2] = inf, -inf, float("nan"), 3.3e38
    S, C = torch.zeros(n, r, device=DEV), torch.zeros(n, r, device=DEV)
    flora.compress(flora.matrices([(n, m)], grads=[G], states=[S], seeds=[9]), r, flora.BF16, 0.0, 1.0)
    flora.compress(flora.matrices([(n, m)], grads=[clean], states=[C], seeds=[9]), r, flora.BF16, 0.0, 1.0)
    sync()
    A = oracle.compress(np.eye(m), r, 9)
    got = to64(S)
    assert np.array_equal(got[3], np.sign(A[5]) * inf) and np.array_equal(got[70], -np.sign(A[m - 1]) * inf)
    assert np.isnan(got[129]).all()
    assert np.abs(got[149] / (3.3e38 * A[2]) - 1).max() < 1e-2          # (3.3e38 as a bf16 value, off by 2^-9)
    rows = [i for i in range(n) if i not in (3, 70, 129, 149)]
    assert rel_fro(got[rows], to64(C)[rows]) < 2.0 ** -23 * m ** 0.5


# -------------------------------------------------------------- transfer
@pytest.mark.parametrize("n,m,r", [(40, 100, 8), (65, 129, 16), (33, 70, 32), (100, 300, 64),
                                   (50, 257, 128), (70, 512, 256)])
def test_momentum_transfer(n, m, r):
    s_old, s_new = 11 + r, 911 + r
    M0 = rand((n, r), 400 + r)
    M = M0.clone()
    mats = flora.matrices([(n, m)], states=[M], seeds=[s_old], seeds_next=[s_new])
    flora.momentum_transfer(mats, r)
    sync()
    ref = oracle.transfer(to64(M0), m, s_old, s_new)
    assert rel_fro(to64(M), ref) < TOL_F32       # fp32 throughout at every rank


@pytest.mark.parametrize("n,m,r", [(40, 100, 8), (65, 129, 16), (33, 70, 32), (100, 300, 64),
                                   (130, 260, 128), (257, 1030, 256)])
@pytest.mark.parametrize("a,b", [(0.9, 0.1 / 16), (0.0, 1.0), (1.0, -0.5)])
def test_transfer_accumulate(n, m, r, a, b):
    # dst <- a dst + b C A_c^T A_m against the literal n x m composition in fp64
    sc, sm = 4242 + r, 9191 + n
    C = rand((n, r), sc)
    M0 = rand((n, r), sm)
    M = M0.clone()
    Cc = C.clone()
    mats = flora.matrices([(n, m)], states=[C], seeds=[sc], seeds_next=[sm])
    flora.transfer_accumulate(mats, r, a, b, [M])
    sync()
    ref = oracle.transfer_accumulate(to64(M0), to64(Cc), m, sc, sm, a, b)
    assert rel_fro(to64(M), ref) < TOL_F32       # fp32 throughout at every rank
    assert torch.equal(C, Cc)                     # the source is only read


# The transfer's split products at the edges of its pieces: chunks of 1024 columns, tiles of 16 columns, blocks
# of 64 rows, r = 256 with many chunks (a workgroup per chunk) and few (one per slab of T).  Bar: what fp32
# sums of this length may be off, 2^-24 sqrt(m + r), plus the generator's share.
@pytest.mark.parametrize("n,m,r,count", [(1, 1, 64, 1), (63, 15, 128, 2), (65, 17, 256, 1), (64, 1024, 64, 1), (130, 1025, 128, 1),
                                         (129, 2047, 256, 1), (70, 1041, 256, 130), (5, 3000, 64, 3)])
def test_transfer_split_products_at_edges(n, m, r, count):
    S0 = [rand((n, r), 700 + l) for l in range(count)]
    st = [x.clone() for x in S0]
    so, sn = [31 + l for l in range(count)], [9031 + l for l in range(count)]
    flora.momentum_transfer(flora.matrices([(n, m)] * count, states=st, seeds=so, seeds_next=sn), r)
    sync()
    for l in sorted({0, count // 2, count - 1}):
        ref = oracle.transfer(to64(S0[l]), m, so[l], sn[l])
        assert rel_fro(to64(st[l]), ref) < 2.0 ** -24 * (m + r) ** 0.5 + 4e-7, l


# One product of two fp32 values as products of parts: a unit state times T = a b^T (one column).  What is left
# out is at most 2^-24 of the product, the last addition rounds by 2^-24, the five before it by less than that
# together; with parts cut off instead of rounded what is left out reaches 2^-22.  Then sums of a few
# columns, against the same sums of fp32 products in numpy.
@pytest.mark.parametrize("r", [64, 128, 256])
def test_transfer_split_products_round_like_fp32(r):
    def A(seed, m):
        a = torch.empty(m, r, device=DEV)
        assert flora.lib().flora_debug_generate(seed, m, r, a.data_ptr(), None, None) == flora.OK
        sync()
        return a.cpu().numpy()

    def T_of(m, s0, s1):
        unit = torch.eye(r, device=DEV)
        flora.momentum_transfer(flora.matrices([(r, m)], states=[unit], seeds=[s0], seeds_next=[s1]), r)
        sync()
        return to64(unit)

    for s in range(8):
        ref = np.outer(A(5 + s, 1)[0].astype(np.float64), A(99 + s, 1)[0].astype(np.float64))
        assert np.abs(T_of(1, 5 + s, 99 + s) / ref - 1.0).max() < 3 * 2.0 ** -24
    for m in (5, 16, 40, 300):
        a, b = A(7, m), A(8, m)
        ref = a.astype(np.float64).T @ b.astype(np.float64)
        fp32 = np.zeros((r, r), np.float32)
        for j in range(m):
            fp32 += np.outer(a[j], b[j])
        assert rel_fro(T_of(m, 7, 8), ref) < rel_fro(fp32, ref), m


# T's tiles dealt to groups of waves: sets around 256 pieces (r = 64 and 128: four and two groups up to there),
# columns around the 64 / 32 of a round there and the 512 / 256 / 128 at r = 8 / 16 / 32.  Same bar.
@pytest.mark.parametrize("n,m,r,count", [(3, 31, 8, 2), (70, 513, 8, 1), (33, 511, 8, 3), (40, 255, 16, 2), (65, 289, 16, 1), (64, 127, 32, 2),
                                         (31, 1154, 32, 1), (20, 63, 64, 256), (20, 65, 64, 257), (9, 31, 128, 256), (9, 33, 128, 257)])
def test_transfer_tiles_in_groups(n, m, r, count):
    test_transfer_split_products_at_edges(n, m, r, count)


# T in blocks, by how many pieces a launch has: either side of every change of block, columns around the 16 of a
# tile and the 128 / 64 of a round of eight / four groups, two pieces per matrix.  Same bar.
@pytest.mark.parametrize("n,m,r,count", [(70, 127, 64, 64), (3, 129, 64, 65), (65, 1040, 128, 8), (20, 65, 128, 17), (9, 63, 128, 65),
                                         (64, 129, 256, 4), (33, 1025, 256, 2), (5, 65, 256, 5), (20, 17, 256, 16), (9, 31, 256, 17),
                                         (1, 33, 256, 64), (7, 16, 256, 65), (2, 15, 256, 129)])
def test_transfer_in_blocks_of_T(n, m, r, count):
    test_transfer_split_products_at_edges(n, m, r, count)


# What is not finite in a state stays in its row and comes out as the fp32 product gives it: inf times T's entry
# has that entry's sign, two infinities of opposite signs in one sum are a NaN, a NaN is one in the whole row.
@pytest.mark.parametrize("n,accumulate", [(70, False), (129, True), (64, False), (1, False)])
@pytest.mark.parametrize("r", [8, 64, 128, 256])
def test_transfer_of_states_that_are_not_finite(r, n, accumulate):
    m, inf = 300, float("inf")
    clean = rand((n, r), 77)
    S = clean.clone()
    put = {0: [(3, inf)], 3: [(5, inf)], 31: [(0, -inf)], 33: [(r - 1, inf), (2, 1e30)], 40: [(0, float("nan"))],
           63: [(1, inf), (r - 2, -inf)], 64: [(r - 1, 3.3e38)], n - 1: [(r // 2, -inf)]}
    put = {i: v for i, v in put.items() if i < n}
    for i, entries in put.items():
        for k, v in entries:
            S[i, k] = v
    M, out = S.clone(), torch.zeros((n, r), device=DEV)
    mats = flora.matrices([(n, m)], states=[M], seeds=[5], seeds_next=[6])
    if accumulate:
        flora.transfer_accumulate(mats, r, 0.0, 1.0, [out])
    else:
        flora.momentum_transfer(mats, r)
        out = M
    sync()
    got = to64(out)
    finite = [i for i in range(n) if i not in put]
    if finite:
        assert rel_fro(got[finite], oracle.transfer(to64(clean), m, 5, 6)[finite]) < TOL_F32
    T = oracle.transfer(np.eye(r), m, 5, 6)
    big = np.abs(T) > 1e-5 * np.abs(T).max()          # (the sign of an entry nearer to zero is a matter of rounding)
    for i, entries in put.items():
        infs = [(k, v) for k, v in entries if np.isinf(v)]
        if any(np.isnan(v) for _, v in entries):
            assert np.isnan(got[i]).all(), i
        elif infs:
            signs = np.stack([np.sign(v) * np.sign(T[k]) for k, v in infs])
            sure = np.stack([big[k] for k, _ in infs]).all(axis=0)
            want = np.where((signs == signs[0]).all(axis=0), signs[0] * inf, np.nan)
            assert np.array_equal(got[i][sure], want[sure], equal_nan=True), i
        else:                                         # huge but finite
            want = entries[0][1] * T[entries[0][0]]
            fits = np.abs(want) < 3e38
            assert fits.any() and np.abs(got[i][fits] / want[fits] - 1).max() < 1e-4


# Two-part products (every matrix of the call has 1024 columns, 2048 at r = 64): rows around the 32 of a block and
# the 64 of an entry, columns around the 32 of a tile, the 1024 of a chunk and the rounds of eight and four groups,
# workgroups whose share of the rows spans matrices (more than 256 entries at r = 256), and states whose rows differ by
# 2^200, a zero row among them.  The bar is that of the other products.
@pytest.mark.parametrize("n,m,r,count", [(1, 2048, 64, 1), (65, 2049, 64, 70), (33, 1024, 128, 1), (130, 1056, 128, 9), (31, 1055, 256, 2),
                                         (64, 2047, 256, 3), (129, 1025, 256, 90), (1700, 1030, 256, 1)])
def test_transfer_two_part_products(n, m, r, count):
    S0 = [rand((n, r), 700 + l) * torch.exp2(torch.arange(n, device=DEV) % 201 - 100.0).view(-1, 1) for l in range(count)]
    for x in S0:
        x[n // 2] = 0
    D0 = [rand((n, r), 900 + l) for l in range(count)]
    st, dst = [x.clone() for x in S0], [x.clone() for x in D0]
    so, sn = [31 + l for l in range(count)], [9031 + l for l in range(count)]
    mats = flora.matrices([(n, m)] * count, states=st, seeds=so, seeds_next=sn)
    flora.transfer_accumulate(mats, r, 0.5, 0.25, dst)
    flora.momentum_transfer(mats, r)
    sync()
    bar = 2.0 ** -24 * (m + r) ** 0.5 + 4e-7
    for l in sorted({0, count // 2, count - 1}):
        ref = oracle.transfer(to64(S0[l]), m, so[l], sn[l])
        got = to64(st[l])
        norms = np.linalg.norm(ref, axis=1)
        assert (np.linalg.norm(got - ref, axis=1) <= 2 * bar * norms).all(), l        # (row by row: twice the bar of a whole)
        sums = 0.5 * to64(D0[l]) + 0.25 * ref
        # (the sum of two terms rounds by 2^-24 of the larger)
        assert (np.abs(to64(dst[l]) - sums) <= 2.0 ** -23 * (np.abs(to64(D0[l])) + np.abs(ref)) + 8 * bar * norms.reshape(-1, 1)).all(), l


# ... wider, and at the widths from which T's own sums take two parts in launches of few chunks (2048 and 2304 columns).
@pytest.mark.parametrize("n,m,r,count", [(40, 2303, 128, 1), (40, 2304, 128, 1), (70, 2048, 128, 12), (33, 5000, 64, 2), (64, 8192, 256, 1), (35, 20011, 64, 1), (9, 70000, 128, 1)])
def test_transfer_two_part_products_of_wide_matrices(n, m, r, count):
    test_transfer_two_part_products(n, m, r, count)


# T as a unit state gets it in a launch of few chunks: no further off than sums of three-part products are (1.09, 1.23 and 1.33e-7
# measured with three parts throughout) and T's second part ends (4.1e-8 in the root mean square), and a twentieth.
@pytest.mark.parametrize("m,three", [(1024, 1.09e-7), (1600, 1.23e-7), (2048, 1.33e-7)])
@pytest.mark.parametrize("r", [128, 256])
def test_transfer_of_a_unit_state_in_short_launches(r, m, three):
    err = size = 0.0
    for k in range(4):
        A = [torch.empty(m, r, device=DEV) for _ in range(2)]
        for a, seed in zip(A, (77 + k, 1077 + k)):
            flora.debug_generate(seed, m, r, a)
        S = torch.eye(r, device=DEV)
        flora.momentum_transfer(flora.matrices([(r, m)], states=[S], seeds=[77 + k], seeds_next=[1077 + k]), r)
        sync()
        T = to64(A[0]).T @ to64(A[1])
        err, size = err + np.sum((to64(S) - T) ** 2), size + np.sum(T ** 2)
    assert (err / size) ** 0.5 < 1.05 * (three ** 2 + 4.1e-8 ** 2) ** 0.5


# ... and states that are not finite there, as above.
@pytest.mark.parametrize("r,m", [(64, 2050), (128, 1030), (256, 1030)])
def test_transfer_two_part_products_of_states_that_are_not_finite(r, m):
    n, inf = 70, float("inf")
    clean = rand((n, r), 77)
    S = clean.clone()
    S[3, 5], S[31, 0], S[40, 2], S[69, r - 1], S[64, 7] = inf, -inf, float("nan"), inf, 3.3e38
    M = S.clone()
    flora.momentum_transfer(flora.matrices([(n, m)], states=[M], seeds=[5], seeds_next=[6]), r)
    sync()
    got, T = to64(M), oracle.transfer(np.eye(r), m, 5, 6)
    finite = [i for i in range(n) if i not in (3, 31, 40, 64, 69)]
    assert rel_fro(got[finite], oracle.transfer(to64(clean), m, 5, 6)[finite]) < TOL_F32
    big = np.abs(T) > 1e-5 * np.abs(T).max()
    for i, k, v in ((3, 5, 1), (31, 0, -1), (69, r - 1, 1)):
        assert np.array_equal(got[i][big[k]], (np.sign(T[k]) * v * inf)[big[k]]), i
    assert np.isnan(got[40]).all()
    want = 3.3e38 * T[7]
    fits = np.abs(want) < 3e38
    # (of the row, not entry by entry: T's own sums over m columns round by 2^-24 sqrt(m) of its size, also where they cancel)
    assert fits.any() and np.linalg.norm((got[64][fits] - want[fits]) / 1e38) < 2e-6 * np.linalg.norm(want[fits] / 1e38)


def test_transfer_accumulate_grouped_and_errors():
    shapes = [(70, 90), (33, 200), (128, 64), (5, 7)]
    r = 16
    C = [rand((n, r), 50 + i) for i, (n, m) in enumerate(shapes)]
    M0 = [rand((n, r), 60 + i) for i, (n, m) in enumerate(shapes)]
    M = [x.clone() for x in M0]
    sc = [int(flora.derive_seed(1, l, 0)) for l in range(len(shapes))]
    sm = [int(flora.derive_seed(2, l, 0)) for l in range(len(shapes))]
    mats = flora.matrices(shapes, states=C, seeds=sc, seeds_next=sm)
    flora.transfer_accumulate(mats, r, 0.5, 0.25, M)
    sync()
    for l, (n, m) in enumerate(shapes):
        ref = oracle.transfer_accumulate(to64(M0[l]), to64(C[l]), m, sc[l], sm[l], 0.5, 0.25)
        assert rel_fro(to64(M[l]), ref) < TOL_F32
    import ctypes
    arr = (ctypes.c_void_p * len(shapes))(*[c.data_ptr() for c in C])       # destination = source
    assert flora.lib().flora_transfer_accumulate(mats, len(shapes), r, 0.5, 0.25, arr, None) == flora.ERR_INVALID
    assert flora.lib().flora_transfer_accumulate(mats, len(shapes), r, 0.5, 0.25, None, None) == flora.ERR_INVALID


# ---------------------------------------------------------------- update
@pytest.mark.parametrize("n,m,r", [(256, 256, 8), (130, 200, 16), (77, 70, 32), (300, 520, 64), (257, 264, 256)])
def test_apply_update_sgd(n, m, r):
    seed = 5000 + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1)
    W = W0.clone()
    st = S.clone()
    mats = flora.matrices([(n, m)], weights=[W], states=[st], seeds=[seed])
    lr, alpha = 0.5, 0.25
    flora.apply_update(mats, r, flora.F32, flora.sgd_update(lr, alpha, zero_state_after=True))
    sync()
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    ref = oracle.sgd(to64(W0), Gt, lr)
    # the update itself must meet the bar, not only W (which it barely changes)
    assert rel_fro(to64(W) - to64(W0), ref - to64(W0)) < update_bar(r, ref, to64(W0))
    assert rel_fro(to64(W), ref) < (1e-6 if r <= 32 else 2e-3)
    assert float(st.abs().max()) == 0.0


@pytest.mark.parametrize("n,m,r", [(130, 200, 16), (300, 520, 64), (257, 264, 256)])
@pytest.mark.parametrize("clip_d,beta2", [(0.0, 0.0), (1.0, 0.0), (0.3, 0.8)])
def test_apply_update_factored(n, m, r, clip_d, beta2):
    seed = 6000 + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1)
    R0 = (rand((n,), seed + 2).abs() + 0.1).contiguous()
    K0 = (rand((m,), seed + 3).abs() + 0.1).contiguous()
    W, R, K = W0.clone(), R0.clone(), K0.clone()
    mats = flora.matrices([(n, m)], weights=[W], states=[S], row_stats=[R], col_stats=[K], seeds=[seed])
    lr, alpha, eps1 = 0.01, 0.5, 1e-30
    flora.apply_update(mats, r, flora.F32, flora.factored_update(lr, alpha, beta2, eps1, clip_d))
    sync()
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    Wr, Rr, Kr = oracle.factored_update(to64(W0), Gt, to64(R0), to64(K0), beta2, eps1, clip_d, lr)
    tol = tol_for(r)
    assert rel_fro(to64(R), Rr) < tol
    assert rel_fro(to64(K), Kr) < tol
    assert rel_fro(to64(W) - to64(W0), Wr - to64(W0)) < update_bar(r, Wr, to64(W0))


# the passes that write n x m arrays at ranks <= 32: one row tile (nothing to fetch ahead), its edges, two and several, in
# row blocks of one and of two tiles; rows on and off line boundaries (launches of fewer workgroups per compute unit)
@pytest.mark.parametrize("rows", [32, 64])
@pytest.mark.parametrize("m", [128, 131])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("r", [8, 16, 32])
def test_written_tiles_at_small_ranks(r, n, m, rows):
    seed = 7300 + 10 * n + r
    S, W0, V0 = rand((n, r), seed), rand((n, m), seed + 1, scale=0.1), (rand((n, m), seed + 2).abs() + 0.1).contiguous()
    guard = torch.full((4, n + 2, m), 7.0, device=DEV)
    out, Ws, Wu, V = (guard[i, 1:n + 1] for i in range(4))
    if m % 4 == 0:                                # (arrays start on 16-byte boundaries)
        Ws.copy_(W0), Wu.copy_(W0), V.copy_(V0)
    else:
        out, Ws, Wu, V, guard = torch.empty_like(W0), W0.clone(), W0.clone(), V0.clone(), None
    Wb = W0.to(torch.bfloat16)
    Wb0 = Wb.clone()
    lr, alpha, beta2, eps1 = 0.5, 0.5, 0.8, 1e-30
    one = lambda **kw: flora.matrices([(n, m)], states=[S], seeds=[seed], **kw)
    flora.set_tuning("decompress_rows", rows)
    try:
        flora.decompress(one(), r, alpha, [out], flora.F32)
        flora.apply_update(one(weights=[Ws]), r, flora.F32, flora.sgd_update(lr, alpha))
        flora.apply_update(one(weights=[Wb]), r, flora.BF16, flora.sgd_update(lr, alpha))
        flora.apply_update(one(weights=[Wu], second_moments=[V]), r, flora.F32, flora.unfactored_update(lr, alpha, beta2, eps1, 1.0))
        sync()
    finally:
        flora.set_tuning("decompress_rows", 0)
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    assert rel_fro(to64(out), Gt) < TOL_F32
    Wr = oracle.sgd(to64(W0), Gt, lr)
    assert rel_fro(to64(Ws) - to64(W0), Wr - to64(W0)) < update_bar(r, Wr, to64(W0))
    assert rel_fro(to64(Wb), oracle.sgd(to64(Wb0), Gt, lr)) < 2.0 ** -9       # one rounding of the result
    Wr, Vr = oracle.adafactor_step(to64(W0), Gt, V=to64(V0), beta2=beta2, eps1=eps1, clip_d=1.0, step=lr, scale_parameter=False)
    assert rel_fro(to64(V), Vr) < TOL_F32
    assert rel_fro(to64(Wu) - to64(W0), Wr - to64(W0)) < update_bar(r, Wr, to64(W0))
    if guard is not None:
        assert float((guard[:, 0] - 7).abs().max()) == 0 and float((guard[:, -1] - 7).abs().max()) == 0


# fp32 rows off line boundaries in launches on either side of 1024 workgroups, from where on a decompression at ranks <= 32
# keeps its waves in step and launches take fewer workgroups per compute unit (decompression at ranks <= 16, plain
# updates at r = 128): the same bits for the same matrices
@pytest.mark.parametrize("r", [8, 16, 32, 128])
def test_many_ragged_matrices(r):
    n, m, count = 40, 515, 208
    assert len(flora.debug_work_items(1, [(n, m)] * count, r)[0]) >= 1024 > len(flora.debug_work_items(1, [(n, m)] * 100, r)[0])
    S, W0 = rand((count, n, r), 7400), rand((count, n, m + 1), 7401)
    W0 = W0.view(count, -1)[:, :n * m].reshape(count, n, m)
    got = []
    for step in (count, 100):
        W, out = [w.clone() for w in W0], [torch.full((n, m), float("nan"), device=DEV) for _ in range(count)]
        for l in range(0, count, step):
            part = range(l, min(l + step, count))
            mats = flora.matrices([(n, m)] * len(part), weights=[W[i] for i in part], states=[S[i] for i in part], seeds=[50 + i for i in part])
            flora.apply_update(mats, r, flora.F32, flora.sgd_update(0.5, 0.5))
            flora.decompress(mats, r, 0.5, [out[i] for i in part], flora.F32)
        sync()
        got.append(W + out)
    assert all(torch.equal(x, y) for x, y in zip(*got))
    for i in (0, 101, count - 1):
        Gt = oracle.decompress(to64(S[i]), m, 50 + i, alpha=0.5)
        assert rel_fro(to64(got[0][count + i]), Gt) < tol_for(r)
        Wr = oracle.sgd(to64(W0[i]), Gt, 0.5)
        assert rel_fro(to64(got[0][i]) - to64(W0[i]), Wr - to64(W0[i])) < update_bar(r, Wr, to64(W0[i]))


# a decompression writes the same bits with and without the non-temporal hint, in every kernel: ranks <= 32, 4 and 16
# bytes per lane, rows on and off line boundaries
@pytest.mark.parametrize("n,m,r", [(70, 96, 16), (70, 101, 32), (70, 192, 64), (65, 101, 64), (70, 128, 128), (33, 260, 256)])
def test_decompress_streamed_output(n, m, r):
    S = rand((n, r), 7200 + r)
    for dtype, fd in ((torch.float32, flora.F32), (torch.bfloat16, flora.BF16)):
        outs = []
        for policy in (1, 3):
            out = torch.full((n, m), float("nan"), device=DEV, dtype=dtype)
            flora.set_tuning("update_wpolicy", policy)
            try:
                flora.decompress(flora.matrices([(n, m)], states=[S], seeds=[r]), r, 0.5, [out], fd)
                sync()
            finally:
                flora.set_tuning("update_wpolicy", 0)
            outs.append(out)
        assert torch.equal(outs[0], outs[1])
        assert rel_fro(to64(outs[0]), oracle.decompress(to64(S), m, r, alpha=0.5)) < (TOL_BF16 if r >= 64 or fd == flora.BF16 else tol_for(r))


# the update kernel for whole lines of bf16 weights: edges of its 32-row blocks and 64-column waves, one and several
# workgroups per row, one and several row blocks, with plain accesses and with the streamed ones of large sets of whole
# lines (the same bits).  The result is rounded to bf16 (2^-9 of a value at most).
@pytest.mark.parametrize("rows", [0, 64])
@pytest.mark.parametrize("n,m,r", [(33, 8, 64), (300, 520, 64), (257, 264, 128), (96, 1096, 128), (65, 72, 256), (200, 1024, 256)])
def test_update_of_whole_bf16_lines(n, m, r, rows):
    seed = 7100 + n + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1).to(torch.bfloat16)
    R0 = (rand((n,), seed + 2).abs() + 0.1).contiguous()
    K0 = (rand((m,), seed + 3).abs() + 0.1).contiguous()
    lr, alpha, eps1, beta2, clip_d = 0.5, 0.5, 1e-30, 0.8, 0.3
    got = []
    flora.set_tuning("decompress_vec", 3)
    flora.set_tuning("decompress_rows", rows)
    try:
        for policy in (1, 4):
            flora.set_tuning("update_wpolicy", policy)
            guard = torch.full((n + 2, m), 7.0, device=DEV, dtype=torch.bfloat16)
            Ws, Wf, R, K = guard[1:n + 1], W0.clone(), R0.clone(), K0.clone()
            Ws.copy_(W0)
            ss = torch.zeros(4, device=DEV)
            mats = flora.matrices([(n, m)], weights=[Ws], states=[S], seeds=[seed])
            assert flora.debug_access_policy(mats, r, flora.BF16, flora.sgd_update(lr, alpha)) == (policy - 1, policy - 1, 0, 1)
            flora.apply_update(mats, r, flora.BF16, flora.sgd_update(lr, alpha))
            flora.apply_update(flora.matrices([(n, m)], weights=[Wf], states=[S], row_stats=[R], col_stats=[K],
                                              seeds=[seed], weight_sumsqs=[ss]), r, flora.BF16,
                               flora.factored_update(lr, alpha, beta2, eps1, clip_d))
            sync()
            got.append((guard, Wf, R, K, ss))
    finally:
        flora.set_tuning("decompress_vec", 0)
        flora.set_tuning("decompress_rows", 0)
        flora.set_tuning("update_wpolicy", 0)
    assert all(torch.equal(x, y) for x, y in zip(*got))
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    assert rel_fro(to64(Ws), oracle.sgd(to64(W0), Gt, lr)) < TOL_BF16 + 2.0 ** -9
    assert float((guard[0] - 7).abs().max()) == 0 and float((guard[-1] - 7).abs().max()) == 0
    Wr, _, _ = oracle.factored_update(to64(W0), Gt, to64(R0), to64(K0), beta2, eps1, clip_d, lr)
    assert rel_fro(to64(Wf), Wr) < TOL_BF16 + 2.0 ** -9
    assert float(ss[0]) == pytest.approx(float((to64(Wf) ** 2).sum()), rel=1e-5)


# both bf16 decompress kernels (4-byte and 16-byte accesses per lane), with one and with several
# row blocks per matrix (which changes how the column statistics are combined), every mode
@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("rows", [0, 64])
@pytest.mark.parametrize("n,m,r", [(300, 520, 64), (257, 264, 256), (200, 1028, 128)])
def test_bf16_decompress_kernels_every_mode(n, m, r, rows, vec):
    seed = 7000 + n + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1)
    R0 = (rand((n,), seed + 2).abs() + 0.1).contiguous()
    K0 = (rand((m,), seed + 3).abs() + 0.1).contiguous()
    lr, alpha, eps1, beta2, clip_d = 0.01, 0.5, 1e-30, 0.8, 0.3
    out32 = torch.full((n, m), float("nan"), device=DEV)
    out16 = torch.full((n, m), float("nan"), device=DEV, dtype=torch.bfloat16)
    Ws, Wf, R, K = W0.clone(), W0.clone(), R0.clone(), K0.clone()
    flora.set_tuning("decompress_vec", vec)
    flora.set_tuning("decompress_rows", rows)
    try:
        flora.decompress(flora.matrices([(n, m)], states=[S], seeds=[seed]), r, alpha, [out32], flora.F32)
        flora.decompress(flora.matrices([(n, m)], states=[S], seeds=[seed]), r, alpha, [out16], flora.BF16)
        flora.apply_update(flora.matrices([(n, m)], weights=[Ws], states=[S], seeds=[seed]), r, flora.F32,
                           flora.sgd_update(lr, alpha))
        flora.apply_update(flora.matrices([(n, m)], weights=[Wf], states=[S], row_stats=[R], col_stats=[K],
                                          seeds=[seed]), r, flora.F32,
                           flora.factored_update(lr, alpha, beta2, eps1, clip_d))
        sync()
    finally:
        flora.set_tuning("decompress_vec", 0)
        flora.set_tuning("decompress_rows", 0)
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    assert rel_fro(to64(out32), Gt) < TOL_BF16
    assert rel_fro(to64(out32), Gt) < 6e-3
    assert rel_fro(to64(out16), Gt) < TOL_BF16
    # row by row and column by column: a misplaced tile would hide in the norm of the whole
    d = to64(out32) - Gt
    assert (np.linalg.norm(d, axis=1) / np.linalg.norm(Gt, axis=1)).max() < TOL_BF16
    assert (np.linalg.norm(d, axis=0) / np.linalg.norm(Gt, axis=0)).max() < TOL_BF16
    assert rel_fro(to64(Ws) - to64(W0), oracle.sgd(to64(W0), Gt, lr) - to64(W0)) < TOL_BF16
    Wr, Rr, Kr = oracle.factored_update(to64(W0), Gt, to64(R0), to64(K0), beta2, eps1, clip_d, lr)
    assert rel_fro(to64(R), Rr) < TOL_BF16
    assert rel_fro(to64(K), Kr) < TOL_BF16
    assert rel_fro(to64(Wf) - to64(W0), Wr - to64(W0)) < TOL_BF16


# ---------------------------------------------------- algorithms end to end
def test_algorithm1_config1_end_to_end():
    wl = workloads.workload(1)
    (n, m), r, tau = wl.shapes[0], wl.r, wl.tau
    gen = workloads.make_generator(wl.seed)
    W0 = workloads.make_weight(n, m, gen).to(DEV)
    Gs = [workloads.make_grad(wl, n, m, gen).to(DEV) for _ in range(tau)]
    gseed = 0
    seed = flora.derive_seed(gseed, 0, 0)
    W = W0.clone()
    C = torch.zeros((n, r), device=DEV)
    for G in Gs:
        flora.compress(flora.matrices([(n, m)], grads=[G], states=[C], seeds=[seed]), r, flora.F32)
    Csnap = C.clone()
    flora.apply_update(flora.matrices([(n, m)], weights=[W], states=[C], seeds=[seed]), r, flora.F32,
                       flora.sgd_update(wl.lr, 1.0 / tau, zero_state_after=True))
    sync()
    Wr, Gt, Cr = oracle.algorithm1_cycle([to64(W0)], [[to64(G)] for G in Gs], r, gseed, 0, wl.lr)
    assert rel_fro(to64(Csnap), Cr[0]) < TOL_F32
    assert rel_fro(to64(W) - to64(W0), Wr[0] - to64(W0)) < update_bar(r, Wr[0], to64(W0))
    assert float(C.abs().max()) == 0.0


@pytest.mark.parametrize("r,gdt", [(16, "f32"), (64, "bf16")])
def test_algorithm2_with_transfers_small(r, gdt):
    shapes = [(96, 160), (40, 264)]
    beta, kappa, steps, lr, gseed = 0.9, 3, 7, 1e-2, 123
    tdt = torch.float32 if gdt == "f32" else torch.bfloat16
    fdt = flora.F32 if gdt == "f32" else flora.BF16
    W0 = [rand(s, 700 + l) for l, s in enumerate(shapes)]
    W = [w.clone() for w in W0]
    M = [torch.zeros((n, r), device=DEV) for n, _ in shapes]
    orc = oracle.Algorithm2(shapes, r, beta, kappa, gseed)
    Wr = [to64(w) for w in W0]
    epoch = [0] * len(shapes)
    seeds = [flora.derive_seed(gseed, l, 0) for l in range(len(shapes))]
    upd = flora.sgd_update(lr, 1.0)
    for t in range(steps):
        Gs = [rand(s, 800 + 10 * t + l, tdt) for l, s in enumerate(shapes)]
        resample = t % kappa == 0
        nxt = list(seeds)
        if resample:
            epoch = [e + 1 for e in epoch]
            nxt = [flora.derive_seed(gseed, l, epoch[l]) for l in range(len(shapes))]
        mats = flora.matrices(shapes, grads=Gs, weights=W, states=M, seeds=seeds, seeds_next=nxt)
        flora.fused_step(mats, r, fdt, flora.F32, beta, 1.0 - beta, resample, upd)
        seeds = nxt
        sync()
        _, Wr = orc.step([to64(g) for g in Gs], Wr, lr)
    tol = tol_for(r)
    for l in range(len(shapes)):
        assert rel_fro(to64(M[l]), orc.M[l]) < tol
        assert rel_fro(to64(W[l]) - to64(W0[l]), Wr[l] - to64(W0[l])) < update_bar(r, Wr[l], to64(W0[l]))
    assert orc.transfers == 3 * len(shapes)


# ---------------------------------------------------------- error returns
def test_error_codes_launch_nothing():
    n, m, r = 16, 16, 16
    G, S = rand((n, m), 1), torch.zeros((n, r), device=DEV)
    L = flora.lib()
    mats = flora.matrices([(n, m)], grads=[G], states=[S], seeds=[1])
    assert L.flora_compress(mats, 1, 12, flora.F32, 1.0, 1.0, None) == flora.ERR_UNSUPPORTED
    assert L.flora_compress(mats, 1, 512, flora.BF16, 1.0, 1.0, None) == flora.ERR_UNSUPPORTED
    assert L.flora_compress(mats, -1, 16, flora.F32, 1.0, 1.0, None) == flora.ERR_INVALID
    assert L.flora_compress(mats, 0, 16, flora.F32, 1.0, 1.0, None) == flora.OK
    bad = flora.matrices([(n, m)], grads=[G.data_ptr() + 4], states=[S], seeds=[1])
    assert L.flora_compress(bad, 1, 16, flora.F32, 1.0, 1.0, None) == flora.ERR_INVALID
    sync()
    assert float(S.abs().max()) == 0.0


def test_more_matrices_than_one_launch_carries_seeds_for():
    # seeds ride in the kernel arguments, 448 per launch: 500 matrices take two launches
    count, n, m, r = 500, 16, 24, 8
    G = rand((count * n, m), 21)
    S = torch.zeros((count * n, r), device=DEV)
    Gs = [G[l * n:(l + 1) * n] for l in range(count)]
    Ss = [S[l * n:(l + 1) * n] for l in range(count)]
    seeds = [1000 + l for l in range(count)]
    flora.compress(flora.matrices([(n, m)] * count, grads=Gs, states=Ss, seeds=seeds), r, flora.F32)
    sync()
    for l in (0, 1, 447, 448, 449, 499):
        assert rel_fro(to64(Ss[l]), oracle.compress(to64(Gs[l]), r, seeds[l])) < TOL_F32
    out = torch.zeros((count * n, m), device=DEV)
    outs = [out[l * n:(l + 1) * n] for l in range(count)]
    flora.decompress(flora.matrices([(n, m)] * count, states=Ss, seeds=seeds), r, 1.0, outs, flora.F32)
    sync()
    for l in (0, 447, 448, 499):
        assert rel_fro(to64(outs[l]), oracle.decompress(to64(Ss[l]), m, seeds[l])) < TOL_F32


@pytest.mark.parametrize("r,gdt", [(16, "f32"), (64, "bf16")])
def test_micro_batches_accumulated_straight_into_the_momentum(r, gdt):
    # one projection for accumulation and momentum: M <- beta M + ((1-beta)/tau) sum_i G_i A, one
    # compress call per micro-batch, against Algorithm 2's EMA line on the exact mean gradient
    n, m, tau, beta, seed = 200, 328, 4, 0.9, 321
    dt = torch.float32 if gdt == "f32" else torch.bfloat16
    G = [rand((n, m), 700 + i, dtype=dt) for i in range(tau)]
    M0 = rand((n, r), 710)
    M = M0.clone()
    for i in range(tau):
        mats = flora.matrices([(n, m)], grads=[G[i]], states=[M], seeds=[seed])
        flora.compress(mats, r, flora.F32 if gdt == "f32" else flora.BF16, beta if i == 0 else 1.0,
                       (1.0 - beta) / tau)
    sync()
    mean = sum(to64(g) for g in G) / tau
    ref = oracle.compress(mean, r, seed, state=to64(M0), a=beta, b=1.0 - beta)
    assert rel_fro(to64(M) - beta * to64(M0), ref - beta * to64(M0)) < tol_for(r)


# More pointer sets than a plan keeps descriptor images of (64 above four matrices, 512 up to there): slots are used
# again while earlier calls are still queued, twice over, and every call must have seen its own pointers.
@pytest.mark.parametrize("count,sets", [(5, 150), (1, 1100)])
def test_more_pointer_sets_than_descriptor_images(count, sets):
    n, m, r = 17, 40, 8
    G = rand((sets, count, n, m), 41)
    st = torch.zeros((sets, count, n, r), device=DEV)
    seeds = [3 + l for l in range(count)]
    mats = [flora.matrices([(n, m)] * count, grads=[G[i, l] for l in range(count)], states=[st[i, l] for l in range(count)], seeds=seeds)
            for i in range(sets)]
    busy = torch.randn(4096, 4096, device=DEV)
    sync()
    for _ in range(2):
        for _ in range(3):
            busy @ busy
        for i in range(sets):
            flora.compress(mats[i], r, flora.F32, 0.5, 1.0)
    sync()
    for i in sorted({0, 1, 63, 64, 65, 127, 128, 149, 511, 512, 513, 1024, sets - 1} & set(range(sets))):
        for l in range(count):
            assert rel_fro(to64(st[i, l]), 1.5 * oracle.compress(to64(G[i, l]), r, seeds[l])) < TOL_F32, (i, l)


def test_a_new_pointer_set_waits_for_an_old_upload_not_for_the_stream():
    count, n, m, r = 5, 16, 32, 8
    G, st = rand((65, count, n, m), 42), torch.zeros((65, count, n, r), device=DEV)
    mats = [flora.matrices([(n, m)] * count, grads=list(G[i]), states=list(st[i]), seeds=list(range(count))) for i in range(65)]
    busy = torch.randn(8192, 8192, device=DEV)
    busy @ busy
    flora.set_tuning("compress_f32_mt", 0)            # plans start anew
    sync()
    for _ in range(3):
        busy @ busy                                   # 1.1 TFLOP each: the uploads below wait for these
    for i in range(64):
        flora.compress(mats[i], r, flora.F32, 0.0, 1.0)
    for _ in range(40):
        busy @ busy
    after = torch.cuda.Event()
    after.record()
    flora.compress(mats[64], r, flora.F32, 0.0, 1.0)  # takes the first one's slot
    assert not after.query()
    sync()
    for i in (0, 63, 64):
        assert rel_fro(to64(st[i, 0]), oracle.compress(to64(G[i, 0]), r, 0)) < TOL_F32

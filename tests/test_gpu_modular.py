"""Products on the int8 matrix cores by residues and sub-digits, whatever the digit width.

Every limb must equal that of the FP64 level products (MDGEMM_STAGED), which the other
GPU tests pin against the oracle; some of these products are checked against the oracle
directly.  The results are roundings of exact integers, so the comparison is bit for bit.
The sizes cover the edges of the 256 x 256 tiles, of the 128-byte k stages and of the
rows of four that the planes hold; the options cover every sub-digit count, residue
systems of one to three limb chunks, and the word counts of the accumulation.
"""

import time

import numpy as np
import pytest
import torch

from oracle import pipeline
from paper_2607_06881_amd import mdgemm as md
from paper_2607_06881_amd import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda"

ALL = md.MDGEMM_CUTOFF_ALL


def _modular(m, n, k, L, **opts):
    """True when the library takes the int8 products (their workspace differs)."""
    flags = opts.pop("flags", 0)
    return (md.mdgemm_workspace_bytes(m, n, k, L, flags=flags | md.MDGEMM_WORKSPACE_SCRATCH, **opts)
            != md.mdgemm_workspace_bytes(m, n, k, L, flags=flags, **opts))


def _operands(L, m, n, k, seed, spread=0):
    rng = np.random.default_rng(seed)
    A = workloads.make_operand(rng, L, m, k, "normal", row_exp=20, elem_exp=spread)
    B = workloads.make_operand(rng, L, k, n, "normal", col_exp=20, elem_exp=spread)
    A[:, 0, :] = 0.0  # an all-zero line of each operand, and single zeros
    if n > 1:
        B[:, :, n - 1] = 0.0
    A[:, m - 1, k // 2] = 0.0
    return torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)


CASES = [
    # limbs, m, n, k, options
    (2, 255, 257, 127, {}),
    (2, 256, 512, 128, {}),
    (2, 257, 511, 129, {}),
    (2, 513, 258, 1, {}),
    (2, 301, 303, 640, {"cutoff": ALL}),
    (1, 511, 301, 260, {}),
    (3, 259, 300, 257, {}),
    (3, 300, 260, 130, {"cutoff": ALL}),
    (4, 262, 290, 200, {}),
    (4, 300, 300, 100, {"cutoff": ALL}),
    (8, 258, 300, 70, {}),
    (16, 258, 264, 40, {}),
    (2, 300, 300, 300, {"range_bits": 60}),
    (2, 300, 300, 300, {"slice_bits": -1}),
    (2, 1500, 1500, 100, {"slice_bits": 22}),
    (3, 700, 700, 200, {"slice_bits": 21, "cutoff": ALL}),
    (2, 300, 300, 90, {"slice_bits": 20}),
    (2, 300, 300, 90, {"slice_bits": 7, "slices": 16}),
    (1, 300, 300, 90, {"slice_bits": 5}),
    (2, 300, 300, 200, {"flags": md.MDGEMM_KARATSUBA}),
    (2, 300, 300, 200, {"cutoff": 3}),
    (2, 70, 4000, 300, {}),
    (2, 4100, 40, 300, {}),
    # a level's pairs split into several sums, more than 264 planes, two GEMM launches
    (16, 300, 300, 1500, {}),
    (8, 300, 300, 4096, {"cutoff": ALL}),
    (8, 300, 300, 7000, {}),
    (4, 258, 260, 16384, {"slice_bits": -1}),
    (2, 300, 300, 5000, {"slice_bits": -1, "range_bits": 60}),
    (11, 300, 270, 60, {"slice_bits": -1}),
    # the longest sums of residues and of sub-digits
    (2, 260, 270, 32768, {}),
    (2, 257, 300, 65536, {"slice_bits": 8}),
]


@pytest.mark.parametrize("L,m,n,k,opts", CASES)
def test_limbs_equal_the_fp64_level_products(L, m, n, k, opts):
    print(f"[case] L={L} {m}x{n}x{k} {opts}", flush=True)
    assert _modular(m, n, k, L, **opts)
    A, B = _operands(L, m, n, k, 5 * m + k, spread=6)
    plain = {x: y for x, y in opts.items() if x != "flags"}
    want = md.mdgemm_ex(A, B, flags=md.MDGEMM_STAGED, **plain)
    got = md.mdgemm_ex(A, B, **opts)
    assert torch.equal(got, want)


@pytest.mark.parametrize("L,m,n,k,opts", [(2, 300, 700, 500, {}), (3, 600, 500, 300, {}),
                                          (3, 513, 600, 200, {"slice_bits": 5}), (2, 400, 400, 300, {"range_bits": 40})])
def test_int8_digits(L, m, n, k, opts):
    """MDGEMM_INT8 chooses the digits; their products equal the FP64 path's at those digits."""
    print(f"[case] int8 digits L={L} {m}x{n}x{k} {opts}", flush=True)
    assert _modular(m, n, k, L, flags=md.MDGEMM_INT8, **opts)
    A, B = _operands(L, m, n, k, 7 * m, spread=4)
    w, S, T = md.mdgemm_plan(m, n, k, L, flags=md.MDGEMM_INT8, **opts)
    want = md.mdgemm_ex(A, B, slice_bits=w, slices=S, cutoff=T, flags=md.MDGEMM_STAGED)
    assert torch.equal(md.mdgemm_ex(A, B, flags=md.MDGEMM_INT8, **opts), want)


@pytest.mark.parametrize("L,m,n,k,opts", [(2, 260, 258, 130, {}), (4, 257, 300, 33, {"cutoff": ALL})])
def test_limbs_equal_the_oracle(L, m, n, k, opts):
    print(f"[case] oracle L={L} {m}x{n}x{k} {opts}", flush=True)
    assert _modular(m, n, k, L, **opts)
    A, B = _operands(L, m, n, k, 11)
    got = md.mdgemm_ex(A, B, **opts).cpu().numpy()
    _, S, T = md.mdgemm_plan(m, n, k, L, **opts)
    rows = [0, 1, m // 2, m - 2, m - 1]
    ref = pipeline.full_reference(A.cpu().numpy()[:, rows], B.cpu().numpy(), S, T)["C"]
    assert np.array_equal(got[:, rows], ref)


@pytest.mark.parametrize("m,n,k,opts", [(260, 258, 512, {}), (260, 258, 512, {"cutoff": ALL}),
                                        (260, 258, 512, {"slice_bits": 20}), (1000, 1000, 400, {"slice_bits": 21}),
                                        # the longest sums of residues (2^15 terms) and of sub-digits (2^16)
                                        (260, 258, 32768, {}), (260, 258, 32768, {"cutoff": ALL}),
                                        (260, 258, 65536, {"slice_bits": 8})])
def test_largest_digits_of_either_sign(m, n, k, opts):
    """Every digit at its largest magnitude: the sums reach their bounds."""
    print(f"[case] largest digits {m}x{n}x{k} {opts}", flush=True)
    A = np.full((2, m, k), 1.0 - 2.0 ** -53)
    A[1] = 2.0 ** -54 * (1.0 - 2.0 ** -53)
    B = np.full((2, k, n), 1.0 - 2.0 ** -53)
    B[1] = 2.0 ** -54 * (1.0 - 2.0 ** -53)
    A[:, ::2] *= -1.0
    B[:, :, ::3] *= -1.0
    Ag, Bg = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    assert _modular(m, n, k, 2, **opts)
    assert torch.equal(md.mdgemm_ex(Ag, Bg, **opts), md.mdgemm_ex(Ag, Bg, flags=md.MDGEMM_STAGED, **opts))


def test_library_buffer_capture_and_a_small_workspace():
    m, n, k, L = 300, 280, 150, 2
    A, B = _operands(L, m, n, k, 3)
    want = md.mdgemm_ex(A, B, flags=md.MDGEMM_STAGED)
    assert torch.equal(md.mdgemm(A, B), want)  # the library's buffer
    # a workspace that only the FP64 path fits is still taken
    need = md.mdgemm_workspace_bytes(m, n, k, L)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    assert torch.equal(md.mdgemm_ex(A, B, workspace=ws, flags=md.MDGEMM_WORKSPACE_SCRATCH), want)
    full = md.mdgemm_workspace_bytes(m, n, k, L, flags=md.MDGEMM_WORKSPACE_SCRATCH)
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    C = torch.empty_like(want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        md.mdgemm_ex(A, B, C, workspace=ws, flags=md.MDGEMM_WORKSPACE_SCRATCH)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            md.mdgemm_ex(A, B, C, workspace=ws, flags=md.MDGEMM_WORKSPACE_SCRATCH)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        print(f"[case] graph replay {rep}", flush=True)
        A2, B2 = _operands(L, m, n, k, 20 + rep)
        A.copy_(A2)
        B.copy_(B2)
        C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, md.mdgemm_ex(A, B, flags=md.MDGEMM_STAGED))


@pytest.mark.parametrize("L,m,n,k,flags", [
    (8, 300, 280, 150, md.MDGEMM_WORKSPACE_SCRATCH),   # the split's integers in more than 64 KB of LDS
    (16, 260, 270, 40, md.MDGEMM_WORKSPACE_SCRATCH),   # two launches of the products
    (2, 1100, 1300, 200, 0),                           # levels in a readable workspace
    (8, 520, 700, 100, 0),
])
def test_capture_of_every_kernel_form(L, m, n, k, flags):
    A, B = _operands(L, m, n, k, 31)
    ws = torch.empty(md.mdgemm_workspace_bytes(m, n, k, L, flags=flags), dtype=torch.uint8, device=DEV)
    C = torch.empty((L, m, n), dtype=torch.float64, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        md.mdgemm_ex(A, B, C, workspace=ws, flags=flags)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        print(f"[case] L={L} {m}x{n}x{k} flags={flags} graph replay {rep}", flush=True)
        A2, B2 = _operands(L, m, n, k, 40 + rep)
        A.copy_(A2)
        B.copy_(B2)
        C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, md.mdgemm_ex(A, B, flags=md.MDGEMM_STAGED))


def test_memory_for_the_fp64_products_only(monkeypatch):
    """Where the larger workspace of the int8 products does not fit the memory, the product runs in
    the FP64 one (here the allocator's refusal of the larger size is played)."""
    m, n, k, L = 4096, 40, 500, 4
    A, B = _operands(L, m, n, k, 13)
    want = md.mdgemm_ex(A, B, flags=md.MDGEMM_STAGED)
    plain = md.mdgemm_workspace_bytes(m, n, k, L)
    full = md.mdgemm_workspace_bytes(m, n, k, L, flags=md.MDGEMM_WORKSPACE_SCRATCH)
    assert plain < full
    empty = torch.empty

    def limited(*size, **kw):
        if size and size[0] == full:
            raise torch.OutOfMemoryError("played")
        return empty(*size, **kw)

    monkeypatch.setattr(md.torch, "empty", limited)
    assert torch.equal(md.mdgemm_ex(A, B), want)


@pytest.mark.parametrize("L,m,n,k,opts", [
    (2, 1283, 1409, 130, {}), (2, 1100, 900, 257, {"cutoff": ALL}), (3, 1025, 1023, 127, {}),
    (2, 1409, 1283, 300, {"slice_bits": 20}), (2, 1409, 1500, 200, {"slice_bits": 21}),
    (2, 1283, 1300, 200, {"slice_bits": 7}), (8, 520, 700, 100, {}), (2, 900, 1000, 200, {"range_bits": 60}),
    # a last tile of few elements: one to three rows of 1 to 40 columns
    (1, 4097, 1, 256, {}), (1, 4097, 17, 256, {}), (1, 4098, 9, 256, {}), (1, 4099, 40, 256, {}),
    (2, 4097, 33, 384, {}),
    # four sub-digits (the int8 panels fit the digit panels' room at whole stages of k), longer k
    (2, 2550, 2500, 256, {"slice_bits": 21}), (4, 1100, 1000, 2048, {}),
])
def test_a_readable_workspace_holds_digits_and_levels(L, m, n, k, opts):
    """Without MDGEMM_WORKSPACE_SCRATCH the workspace holds the exponents, digit panels and
    level planes of the pair schedule, whichever matrix cores formed the levels: every
    byte of them equals the FP64 path's."""
    print(f"[case] readable workspace L={L} {m}x{n}x{k} {opts}", flush=True)
    A, B = _operands(L, m, n, k, m + n, spread=6)
    lay = md.mdgemm_workspace_layout(m, n, k, L, **opts)
    assert lay["direct_levels"] == 1
    need = md.mdgemm_workspace_bytes(m, n, k, L, **opts)
    ws = [torch.full((need,), fill, dtype=torch.uint8, device=DEV) for fill in (0x5a, 0x33)]
    got = md.mdgemm_ex(A, B, workspace=ws[0], **opts)
    want = md.mdgemm_ex(A, B, workspace=ws[1], flags=md.MDGEMM_STAGED, **opts)
    assert torch.equal(got, want)
    parts = [md.workspace_parts(ws[0], m, n, k, L, **opts),
             md.workspace_parts(ws[1], m, n, k, L, flags=md.MDGEMM_STAGED, **opts)]
    for name in ("EA", "EB", "DA", "DB", "G"):
        assert torch.equal(parts[0][name], parts[1][name]), name
    assert not torch.signbit(parts[0]["G"][parts[0]["G"] == 0]).any().item()


@pytest.mark.parametrize("m,n,k,opts", [
    # 7-bit digits are not split: 15 pairs of 127^2 each pass 2^31 between these two k
    (1024, 1024, 8876, {"slice_bits": 7}), (1024, 1024, 8877, {"slice_bits": 7}),
    (1024, 1024, 9000, {"slice_bits": 7}), (1024, 1024, 24000, {"slice_bits": 6}),
])
def test_levels_of_the_largest_digits_in_a_readable_workspace(m, n, k, opts):
    print(f"[case] largest digits, readable workspace {m}x{n}x{k} {opts}", flush=True)
    A = torch.full((2, m, k), 1.0 - 2.0 ** -53, dtype=torch.float64, device=DEV)
    B = torch.full((2, k, n), 1.0 - 2.0 ** -53, dtype=torch.float64, device=DEV)
    A[1], B[1] = 2.0 ** -54 * (1.0 - 2.0 ** -53), 2.0 ** -54 * (1.0 - 2.0 ** -53)
    A[:, ::2] *= -1.0
    need = md.mdgemm_workspace_bytes(m, n, k, 2, **opts)
    ws = [torch.empty(need, dtype=torch.uint8, device=DEV) for _ in range(2)]
    got = md.mdgemm_ex(A, B, workspace=ws[0], **opts)
    want = md.mdgemm_ex(A, B, workspace=ws[1], flags=md.MDGEMM_STAGED, **opts)
    assert torch.equal(got, want)
    parts = [md.workspace_parts(w, m, n, k, 2, flags=f, **opts) for w, f in zip(ws, (0, md.MDGEMM_STAGED))]
    assert torch.equal(parts[0]["G"], parts[1]["G"])


@pytest.mark.parametrize("L,m,n,k,opts", [(2, 700, 650, 300, {}), (3, 513, 600, 200, {"slice_bits": 5})])
def test_a_readable_int8_workspace_holds_digits_and_levels(L, m, n, k, opts):
    """The parts that the header lists for MDGEMM_INT8, at the sizes where products in scratch run
    otherwise: exponents, A's digits and the int32 levels equal the FP64 path's at those digits."""
    print(f"[case] readable int8 workspace L={L} {m}x{n}x{k} {opts}", flush=True)
    int8 = md.MDGEMM_INT8
    assert _modular(m, n, k, L, flags=int8, **opts)
    A, B = _operands(L, m, n, k, 9 * m, spread=4)
    w, S, T = md.mdgemm_plan(m, n, k, L, flags=int8, **opts)
    need = md.mdgemm_workspace_bytes(m, n, k, L, flags=int8, **opts)
    ws = torch.full((3 * need,), 0x5a, dtype=torch.uint8, device=DEV)  # room for any path
    got = md.mdgemm_ex(A, B, workspace=ws, flags=int8, **opts)
    digits = dict(slice_bits=w, slices=S, cutoff=T, flags=md.MDGEMM_STAGED)
    staged = torch.empty(md.mdgemm_workspace_bytes(m, n, k, L, **digits), dtype=torch.uint8, device=DEV)
    assert torch.equal(got, md.mdgemm_ex(A, B, workspace=staged, **digits))
    want = md.workspace_parts(staged, m, n, k, L, **digits)
    up = lambda x, to: (x + to - 1) // to * to  # noqa: E731
    kp, mp, np_ = up(k, 128), up(m, 256), up(n, 256)
    pitch, off, parts = 128 + S * kp, 0, {}
    for name, size in (("EA", 4 * m), ("EB", 4 * n), ("flag", 4), ("DA", mp * pitch), ("DB", np_ * pitch),
                       ("G", 4 * (T + 1) * m * n)):
        parts[name] = ws[off:off + size]
        off += up(size, 256)
    untouched = bool((ws[need:] == 0x5a).all())  # not in the assert, whose report would walk the tensor
    assert off == need and untouched
    assert torch.equal(parts["EA"].view(torch.int32), want["EA"])
    assert torch.equal(parts["EB"].view(torch.int32), want["EB"])
    da = parts["DA"].view(torch.int8).view(mp, pitch)[:m, 128:].reshape(m, S, kp)[:, :, :k]
    assert torch.equal(da.to(torch.float32), want["DA"][:S, :k, :m].to(torch.float32).permute(2, 0, 1))
    levels = parts["G"].view(torch.int32).view(T + 1, m, n)
    assert md.mdgemm_workspace_layout(m, n, k, L, **digits)["direct_levels"]
    assert torch.equal(levels.to(torch.float64), want["G"])
    # the program may keep other data in the part of its buffer that the call does not need
    C = ws[need:need + 8 * got.numel()].view(torch.float64).view(got.shape)
    assert torch.equal(md.mdgemm_ex(A, B, C, workspace=ws, flags=int8, **opts), got)


def test_stage_times_of_levels_on_int8():
    """The digits that the workspace is left with are split after the accumulation, and count as
    split: the accumulation's own time is that of the FP64 levels' call (the same kernel and planes;
    with the two splits in it, it would be more than four times as long)."""
    m, n, k, opts = 1100, 900, 4096, {"cutoff": ALL}
    print(f"[case] stage times, readable workspace {m}x{n}x{k}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(3)
    A, B = (torch.randn(2, *shape, dtype=torch.float64, device=DEV, generator=g) for shape in ((m, k), (k, n)))
    A[1], B[1] = A[0] * 2.0 ** -55, B[0] * 2.0 ** -55
    ws = torch.empty(md.mdgemm_workspace_bytes(m, n, k, 2, **opts), dtype=torch.uint8, device=DEV)
    times = {}
    for flags in (md.MDGEMM_STAGED, 0):
        calls = []
        for _ in range(4):
            md.mdgemm_ex(A, B, workspace=ws, flags=flags | md.MDGEMM_TIME_STAGES, **opts)
            calls.append(md.mdgemm_stage_times())
        times[flags] = np.min(calls, axis=0)
    staged, int8 = times[md.MDGEMM_STAGED], times[0]
    assert int8[2] < 0.5 * staged[2]  # the levels did run on the int8 matrix cores
    assert int8[3] < 2.0 * staged[3] and int8[1] > staged[1], times


def test_library_buffer_that_cannot_grow():
    """A product whose int8 panels exceed the card's memory runs on FP64 in the library's buffer, which
    is neither freed nor waited for on the way: only the first call takes time on the host."""
    L, m, n, k = 4, 18 << 20, 16, 16
    total = torch.cuda.get_device_properties(0).total_memory
    if md.mdgemm_workspace_bytes(m, n, k, L, flags=md.MDGEMM_WORKSPACE_SCRATCH) < total or total < 200 << 30:
        pytest.skip("the panels fit, or the FP64 ones do not")
    torch.cuda.empty_cache()
    A = torch.zeros(L, m, k, dtype=torch.float64, device=DEV)
    A[0] = 1.5
    A[1] = 2.0 ** -60
    A[0, :, 3] = torch.arange(m, dtype=torch.float64, device=DEV)
    B, _ = _operands(L, k, 2, n, 3)
    host = []
    for rep in range(4):
        print(f"[case] library buffer {m}x{n}x{k}, call {rep}", flush=True)
        torch.cuda.synchronize()
        start = time.perf_counter()
        C = md.mdgemm(A, B)
        host.append(time.perf_counter() - start)
    torch.cuda.synchronize()
    rows = slice(m - 1000, m)
    assert torch.equal(C[:, rows], md.mdgemm_ex(A[:, rows].contiguous(), B, flags=md.MDGEMM_STAGED))
    del A, C
    torch.cuda.empty_cache()
    md.mdgemm_release()
    assert max(host[1:]) < 0.1, host


def _least(total, shapes):
    """A QR's or Taylor series' workspace without room for the int8 products: the size with
    its part for the products (the largest need of `shapes`) replaced."""
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    plain = [md.mdgemm_workspace_bytes(*s, 2, slice_bits=-1) for s in shapes]
    full = [md.mdgemm_workspace_bytes(*s, 2, slice_bits=-1, flags=md.MDGEMM_WORKSPACE_SCRATCH) for s in shapes]
    return total - up(max(plain + full)) + up(max(plain))


def _panels(m, nf, n, nb=64):
    for j0 in range(0, nf, nb):
        jb = min(nb, nf - j0)
        mp, nc = m - j0, n - j0 - jb
        if nc:
            yield from ((jb, nc, mp), (jb, nc, jb), (mp, nc, jb))


@pytest.mark.parametrize("m,n", [(700, 640), (1027, 517), (1030, 1030)])
def test_qr_in_both_workspaces(m, n):
    """The trailing products on either matrix cores: the same factors, bit for bit."""
    need = int(md.lib().mdgemm_qr_dd_workspace_bytes(m, n, 64))
    least = _least(need, list(_panels(m, n, n)))
    print(f"[case] qr {m}x{n}: {need} or {least} bytes", flush=True)
    A, _ = _operands(2, m, 8, n, m + n)
    A[0, 0, :] = 1.0
    A[:, :, n - 1] = A[:, :, 0]
    got = [md.mdgemm_qr_dd(A.clone(), workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
           for size in (need, least)]
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    work, tau, ws = A.clone(), torch.empty(2, n, dtype=torch.float64, device=DEV), torch.empty(need, dtype=torch.uint8, device=DEV)
    assert md.lib().mdgemm_qr_dd(m, n, 64, work.data_ptr(), tau.data_ptr(), ws.data_ptr(), least - 1,
                                 None) == md.MDGEMM_EWORKSPACE
    assert torch.equal(work, A)


@pytest.mark.parametrize("n,r,d", [(300, 20, 3), (513, 64, 2)])
def test_taylor_in_both_workspaces(n, r, d):
    need = int(md.lib().mdgemm_taylor_dd_workspace_bytes(n, r, d))
    qr = list(_panels(n, n, 2 * n))
    own = [(n, r, n)] + [(min(64, n - j), n, n - j - 64) for j in range(0, n - 64, 64)]
    own += [(n, r, k * n) for k in range(1, d + 1)]
    least = _least(_least(need, qr), own)
    print(f"[case] taylor n={n} r={r} d={d}: {need} or {least} bytes", flush=True)
    gen = torch.Generator().manual_seed(n)
    A = torch.randn(d + 1, 2, n, n, dtype=torch.float64, generator=gen)
    A[:, 1] *= 2.0 ** -56
    A[0, 0] += 4 * n ** 0.5 * torch.eye(n, dtype=torch.float64)
    B = torch.randn(d + 1, 2, n, r, dtype=torch.float64, generator=gen)
    B[:, 1] *= 2.0 ** -56
    A, B = A.to(DEV), B.to(DEV)
    got = [md.mdgemm_taylor_dd(A, B, workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
           for size in (need, least)]
    assert torch.isfinite(got[0]).all()
    assert torch.equal(got[0], got[1])

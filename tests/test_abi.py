"""CPU-side checks of the boundary: the library loads, exports every symbol the header declares, the
Python binding declares the same set, and the host-only entry points behave."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2108_01624_amd as pkg
    from paper_2108_01624_amd import build

    if not os.path.exists(build.LIB_PATH) or not os.path.exists(build.NATIVE_PATH):
        build.build_library()
    return pkg.load_library()


def _declared():
    src = open(os.path.join(ROOT, "include", "dpclip.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(dp_[a-z0-9_]+)\s*\(", src)))


def test_header_symbols_are_exported(lib):
    names = _declared()
    assert len(names) >= 17
    for n in names:
        assert hasattr(lib, n), f"{n} declared in dpclip.h but not exported"


def test_binding_matches_header(lib):
    from paper_2108_01624_amd import binding

    assert sorted(binding.SIGNATURES) == _declared()
    for n in _declared():
        assert callable(getattr(binding, n)), n


def test_status_strings(lib):
    from paper_2108_01624_amd import binding

    for code, name in binding.STATUS_NAMES.items():
        assert binding.dp_status_str(code) == name
    assert binding.dp_status_str(-99) == "DP_ERR_UNKNOWN"
    assert binding.dp_last_error(None) == "no context"


def test_choose_path_rule(lib):
    import paper_2108_01624_amd as pkg

    # Gram iff (T+1)/2 * (d_in + d_out) <= d_in * d_out (symmetric Gram flops against materialisation flops)
    assert pkg.dp_choose_path(128, 1024, 1024) == pkg.DP_PATH_GRAM
    assert pkg.dp_choose_path(128, 1024, 4096) == pkg.DP_PATH_GRAM
    assert pkg.dp_choose_path(128, 768, 768) == pkg.DP_PATH_GRAM
    assert pkg.dp_choose_path(512, 1024, 1024) == pkg.DP_PATH_GRAM   # the flop tie goes to the symmetric Gram
    assert pkg.dp_choose_path(512, 1024, 4096) == pkg.DP_PATH_GRAM
    assert pkg.dp_choose_path(512, 128, 128) == pkg.DP_PATH_MATERIALISE
    assert pkg.dp_choose_path(128, 64, 64) == pkg.DP_PATH_MATERIALISE
    assert pkg.dp_choose_path(16, 64, 64, pkg.DP_F32) == pkg.DP_PATH_GRAM
    with pytest.raises(pkg.DpError):
        pkg.dp_choose_path(-1, 4, 4)
    with pytest.raises(pkg.DpError):
        pkg.dp_choose_path(1, 4, 4, 5)


def _unit_cells(word):
    """The cells (r, c), r <= c, of one unit word of dp_gram_unit_plan, and the panels it fills."""
    a, b, c2, blk = word & 255, (word >> 8) & 255, (word >> 16) & 255, (word >> 24) & 1
    if blk:
        assert b == a and c2 == a + 1, hex(word)
        return [(a, a), (a, c2), (c2, c2)], {a, c2}
    cells = [tuple(sorted((a, b)))]
    if c2 != 255:
        cells.append(tuple(sorted((a, c2))))
    return cells, {a, b} | ({c2} if c2 != 255 else set())


@pytest.mark.parametrize("T", [129, 256, 300, 384, 512, 640, 768, 1024, 1100, 1920, 2048])
def test_gram_unit_plan_covers_the_upper_triangle_once(lib, T):
    import paper_2108_01624_amd as pkg

    nblk = -(-T // 128)
    words = pkg.dp_gram_unit_plan(T)
    seen, fills = [], 0
    for w in words:
        cells, panels = _unit_cells(w)
        assert all(0 <= r <= c < nblk for r, c in cells), (hex(w), nblk)
        # what a workgroup's registers hold: a diagonal block, or at most two cells of which only the first may be diagonal
        if not (w >> 24) & 1 and len(cells) == 2:
            assert cells[1][0] != cells[1][1], hex(w)
        assert len(panels) <= 3
        seen += cells
        fills += len(panels)
    want = [(r, c) for r in range(nblk) for c in range(r, nblk)]
    assert sorted(seen) == want                      # every cell of the triangle exactly once
    assert sum(1 for w in words if (w >> 24) & 1) == nblk // 2   # every pair of neighbouring panels forms a diagonal block
    assert sum(1 for w in words if not (w >> 24) & 1 and (w >> 16) & 255 == 255) <= 1  # at most one cell on its own
    if T == 512:
        assert len(words) == 4 and fills == 10
    if T == 256:
        assert len(words) == 1 and fills == 2


def test_gram_unit_plan_rejects_other_lengths(lib):
    import paper_2108_01624_amd as pkg

    for T in (0, 1, 128, 2049, -5):
        with pytest.raises(pkg.DpError):
            pkg.dp_gram_unit_plan(T)
    import ctypes
    buf, n = (ctypes.c_uint32 * 2)(), ctypes.c_int()
    assert lib.dp_gram_unit_plan(512, buf, 2, ctypes.byref(n)) == -7   # 4 units do not fit 2 words
    assert lib.dp_gram_unit_plan(512, None, 2, ctypes.byref(n)) == -1


@pytest.mark.parametrize("rows", [1, 40, 129, 1024, 4096])
@pytest.mark.parametrize("d_in", [1, 32, 64, 1000])
def test_fp32_sum_plan_fits_its_rows_into_32_bits(lib, rows, d_in):
    """The bytes of a block of rows, and the offsets into it, are 32-bit numbers: at any width the block that the plan takes has to
    fit, or the rows are addressed with 64 bits."""
    import paper_2108_01624_amd as pkg

    widths = [4, 1 << 20] + [w + e for w in (1 << 21, 1 << 22, 1 << 23, 1 << 24, 1 << 28) for e in (-1, 0, 1, 31)]
    for w in widths:
        for a, b in ((d_in, w), (min(w, 1 << 21), d_in)):
            plan = pkg.dp_dense_sum_plan(pkg.DP_F32, 1, 1, rows, a, b)
            assert plan["block_rows"] * 4 * max(a, b) < 1 << 32, (a, b, plan)
            assert plan["block_rows"] > 0 or max(a, b) >= 1 << 23, (a, b, plan)
            assert -(-a // plan["tile_m"]) <= 65535, (a, b, plan)


@pytest.mark.parametrize("B,T,d_in,d_out", [(1, 1, 752, 113056), (1, 1, 3496, 3544), (40, 20, 1024, 1024), (33, 1, 256, 4096)])
@pytest.mark.parametrize("n", [1, 5])
def test_scaled_form_is_planned_only_where_its_buffers_fit(lib, n, B, T, d_in, d_out):
    """bf16(c * g) of every layer of a launch, and a bias partial for every run of rows (at most one per 32 rows, at most 256)."""
    import paper_2108_01624_amd as pkg

    K, up, planned = B * T, lambda x: -(-x // 256) * 256, 0
    for pct in range(50, 1300, 5):
        ws = 2048 + 2 * K * d_out * pct // 100
        plan = pkg.dp_dense_sum_plan(pkg.DP_BF16, n, B, T, d_in, d_out, ws)
        if plan["scaled"]:
            planned += 1
            runs = min(256, -(-K // 32), max(1, 2048 // (-(-d_out // 256) * plan["layers"])))
            assert plan["layers"] * (up(2 * K * d_out) + 4 * runs * d_out) <= ws, (ws, plan)
    assert planned


def test_dense_sum_plan_refuses_what_the_call_refuses(lib):
    import paper_2108_01624_amd as pkg

    for bad in ((7, 1, 1, 1, 8, 8), (1, 0, 1, 1, 8, 8), (1, 1, 0, 1, 8, 8), (1, 1, 1, 1, 8, 12), (0, 1, 1 << 16, 1 << 15, 8, 8)):
        with pytest.raises(pkg.DpError):
            pkg.dp_dense_sum_plan(*bad)
    assert lib.dp_dense_sum_plan(0, 1, 1, 1, 8, 8, 0, None) == -1
    # bf16: offsets into a 32-row stage, (31 w + columns up to w + a tile's overhang) * 2 bytes, stay below 2^31
    widest = ((1 << 30) - 256) // 32
    assert (31 * widest + widest + 255) * 2 < 1 << 31 <= (32 * (widest + 8) + 256) * 2
    for a, b in ((8, widest), (widest, 8)):
        plan = pkg.dp_dense_sum_plan(pkg.DP_BF16, 1, 1, 20, a, b, 1 << 34)
        assert not (plan["scaled"] and b > 65535 * 256), plan
        for w in (widest + 8, 1 << 26):
            with pytest.raises(pkg.DpError):
                pkg.dp_dense_sum_plan(pkg.DP_BF16, 1, 1, 20, w if a > b else a, b if a > b else w)


def test_null_context_is_rejected_without_a_gpu(lib):
    assert lib.dp_sync(None) == -1
    assert lib.dp_destroy(None) == -1
    assert lib.dp_zero_f32(None, None, 0) == -1
    assert lib.dp_create(None, None, 0) == -1


def test_manifest_counts():
    import dp_synth as syn

    assert syn.manifest_param_count(syn.CONFIGS["C1"]["manifest"]()) == 4096
    assert syn.manifest_param_count(syn.CONFIGS["C2"]["manifest"]()) == 85_054_464
    assert syn.manifest_param_count(syn.CONFIGS["C3"]["manifest"]()) == 334_088_192


def test_schedules_match_the_oracle(lib):
    """Host-only entry points (no GPU work): every step of the paper's run, and ragged small cases."""
    import paper_2108_01624_amd as pkg
    from oracle import dp_oracle as orc

    for t in list(range(1, 7600)) + [9999, 19999, 20000, 20001, 1 << 40]:
        assert pkg.dp_batch_size_schedule(t, 262144, 1048576, 7500, 4) == orc.batch_size_schedule(t, 262144, 1048576, 7500, 4)
    for t in list(range(1, 20003, 7)) + [7499, 7500, 7501, 19999, 20000]:
        got, ref = pkg.dp_lr_schedule(t, 6.0902e-4, 7500, 20000), orc.lr_schedule(t, 6.0902e-4, 7500, 20000)
        assert abs(got - ref) <= 1e-15 * abs(ref)
    for args in ((10, 20, 7, 3), (64, 64, 4, 2), (1, 1000, 13, 13), (5, 6, 100, 7)):
        for t in range(1, 2 * args[2] + 3):
            assert pkg.dp_batch_size_schedule(t, *args) == orc.batch_size_schedule(t, *args)
    for bad in ((0, 1, 2, 4, 2), (1, 1, 2, 4, 0), (1, 3, 2, 4, 2), (1, 1, 2, 1, 2)):
        with pytest.raises(pkg.DpError):
            pkg.dp_batch_size_schedule(*bad)
    with pytest.raises(pkg.DpError):
        pkg.dp_lr_schedule(0, 1e-3, 10, 20)
    with pytest.raises(pkg.DpError):
        pkg.dp_lr_schedule(1, 1e-3, 30, 20)


def test_privacy_accounting_matches_the_oracle(lib):
    """Host-only entry points: log-space double arithmetic against the oracle's 60-digit term-by-term sum."""
    import math

    import paper_2108_01624_amd as pkg
    from oracle import dp_oracle as orc

    for q in (0.0, 1e-6, 7.6e-4, 3.03e-3, 0.05, 0.5, 1.0):
        for sigma in (0.3, 0.6, 1.0, 4.0):
            for alpha in (2, 3, 7, 32, 128, 256):
                got, ref = pkg.dp_rdp_sampled_gaussian(q, sigma, alpha), orc.rdp_sampled_gaussian(q, sigma, alpha)
                assert abs(got - ref) <= 1e-10 * abs(ref) + 1e-16, (q, sigma, alpha, got, ref)
    N = 346_000_000
    q = [262144 / N, 458752 / N, 655360 / N, 851968 / N, 1048576 / N]
    steps = [1875, 1875, 1875, 1875, 12500]
    for sigma in (0.5, 0.6, 1.0):
        got, ref = pkg.dp_rdp_epsilon(q, steps, sigma, 2.89e-9, 64), orc.rdp_epsilon(q, steps, sigma, 2.89e-9, 64)
        assert got[1] == ref[1] and math.isclose(got[0], ref[0], rel_tol=1e-10)
    assert pkg.dp_rdp_epsilon([], [], 1.0, 1e-5, 8)[0] == math.log(1e5) / 7      # no steps: only the conversion term is left
    for bad in ((-0.1, 1.0, 2), (1.1, 1.0, 2), (0.1, 0.0, 2), (0.1, 1.0, 1)):
        with pytest.raises(pkg.DpError):
            pkg.dp_rdp_sampled_gaussian(*bad)
    with pytest.raises(pkg.DpError):
        pkg.dp_rdp_epsilon([0.1], [1], 1.0, 0.0, 8)
    # the noise multiplier for a target: the same search as the oracle's, so the two ends agree to the search tolerance;
    # the result meets the target by the library's own accounting and nothing three tolerances smaller does
    tol = 1e-5
    for target in (2.0, 5.36):
        got = pkg.dp_rdp_noise_multiplier(q, steps, target, 2.89e-9, 32, tol)
        ref = orc.rdp_noise_multiplier(q, steps, target, 2.89e-9, 32, tol)
        assert abs(got - ref) <= 2 * tol * ref, (target, got, ref)
        assert pkg.dp_rdp_epsilon(q, steps, got, 2.89e-9, 32)[0] <= target
        assert pkg.dp_rdp_epsilon(q, steps, got * (1 - 3 * tol), 2.89e-9, 32)[0] > target
    assert pkg.dp_rdp_noise_multiplier([0.1], [0], 1.0, 1e-5, 32, tol) <= 2.0 ** -9      # nothing to protect
    for bad in ((0.0, tol), (1.0, 0.0), (1.0, 1.0), (0.9 * math.log(1 / 2.89e-9) / 31, tol)):    # last: below the conversion term
        with pytest.raises(pkg.DpError):
            pkg.dp_rdp_noise_multiplier(q, steps, bad[0], 2.89e-9, 32, bad[1])


def test_native_calls_leave_alone_what_they_do_not_expect(lib):
    """Another element type, a shape that does not fit, an address in place of a tensor, a closed context: None, and the library is
    not called (there is no context behind the handle given here)."""
    import torch

    from paper_2108_01624_amd import binding

    nat, h = binding._native, 1 << 40
    f, d, A, G = torch.zeros(4), torch.zeros(4, dtype=torch.float64), torch.zeros(2, 3, 8), torch.zeros(2, 3, 16)
    ids, E = torch.zeros(2, 3, dtype=torch.int32), torch.zeros(5, 16)
    H, dL = torch.zeros(2, 4, 16), torch.zeros(2, 4, 5)
    adam = (0, 0.5, 1.0, 1, 1, 8, 1e-3, 0.9, 0.99, 1e-11, 0.0, True)
    for args in ((None, f, None), (0, f, None), (h, d, None), (h, 4096, None), (h, f, -1), (h, f, 2.0), (h, f)):
        assert nat.zero_f32(*args) is None, args
    for args in ((h, A[0], G, True, 0, f), (h, A, G, True, 0, d), (h, A.half(), G, True, 0, f), (h, A, G, True, "auto", f)):
        assert nat.sqnorms_dense(*args) is None
    for a, g in (([A], [G, G]), ([A, A[:1]], [G, G]), ([A], [G[:, :2]]), ([A], [G.bfloat16()]), ((A,), [G]), ([], [])):
        assert nat.sqnorms_dense_batched(h, a, g, True, 0, f) is None
        assert nat.clip_accumulate_dense_batched(h, a, g, 1.0, f, [E] * len(a), None) is None
    assert nat.clip_accumulate_dense_batched(h, [A], [G], 1.0, f, [E.double()], None) is None
    assert nat.clip_accumulate_dense_batched(h, [A], [G], 1.0, f, [E], [f, f]) is None
    assert nat.clip_accumulate_dense(h, A, G, "1", f, E, None) is None
    assert nat.sqnorms_embedding(h, ids.long(), G, 5, False, f) is None
    assert nat.clip_accumulate_embedding(h, ids, G, 2**31, 1.0, f, E) is None
    assert nat.sqnorms_tied_embedding(h, ids, G, H[:, :3], dL, f) is None
    assert nat.clip_accumulate_tied_embedding(h, ids, G, H, dL, 1.0, f, E[:4]) is None
    assert nat.noise_adamw(h, f, f, f, d, 4, *adam) is None
    assert nat.noise_adamw(h, f, f, f, f, 4, *adam[:3], -1, *adam[4:]) is None
    assert nat.noise_adamw(h, f, f, f, f, 4, *adam, f[:1]) is None
    ok = dict(kind="dense", A=A, G=G, has_bias=True)
    for bad in ([], [dict(ok, G=G[:, :2])], [dict(ok, A=A[0])], [dict(ok, G=G.bfloat16())], [{k: v for k, v in ok.items() if k != "has_bias"}],
                [ok, dict(ok, A=A[:1], G=G[:1])], [dict(kind="layernorm", X=A, G=G)], [dict(kind="embedding", ids=ids, G=G, V=5)],
                [dict(kind="embedding", ids=ids[:, :2], G=G, V=5, distinct=False)], (ok,)):
        assert nat.pass1(h, bad, f, {}, None, 2) is None
        assert nat.pass2(h, bad, 1.0, f, E, [[(0, 128), (512, 16)]] * 2, {}, None, 2) is None
    assert nat.pass2(h, [ok], 1.0, f, E, [[(0, 128)]], {}, None, 2) is None


def test_step_runner_refuses_what_the_addresses_cannot_carry():
    """The step driver hands layers over by address: shapes that do not belong together and a sum buffer that cannot hold
    every parameter are refused before the library is called."""
    import torch

    import dp_synth as syn
    import paper_2108_01624_amd as pkg

    class NoCalls:
        handle = None

        def __getattr__(self, name):
            return lambda *a, **k: None

    man = syn.single_dense_manifest(8, 16, True)
    run = pkg.StepRunner(NoCalls(), man, 2, device="cpu")
    A, G = torch.zeros(2, 3, 8), torch.zeros(2, 3, 16)
    layer = lambda a, g: [dict(kind="dense", A=a, G=g, has_bias=True)]
    for bad in (torch.zeros(2, 4, 16), torch.zeros(3, 3, 16)):
        with pytest.raises(ValueError):
            run.pass1(layer(A, bad))
        with pytest.raises(ValueError):
            run.pass2(layer(A, bad), 1.0)
    full = run.S
    for S in (full[:-1], torch.zeros(2 * full.numel())[::2]):
        run.S = S
        with pytest.raises(ValueError):
            run.pass2(layer(A, G), 1.0)
    run.S = full.double()
    with pytest.raises(TypeError):
        run.pass2(layer(A, G), 1.0)


@pytest.mark.parametrize("native", ["missing", "unreadable"])
def test_loading_without_the_extension_says_how_to_build_it(lib, tmp_path, native):
    """A library whose extension is not there, or cannot be loaded, is refused with the instruction that a missing library gets."""
    import shutil
    import subprocess
    import sys

    from paper_2108_01624_amd import build

    top = tmp_path / "paper_2108_01624_amd"
    top.mkdir()
    for f in os.listdir(build.PKG_DIR):
        if f.endswith(".py"):
            shutil.copy(os.path.join(build.PKG_DIR, f), top / f)
    shutil.copy(build.LIB_PATH, top / "libdpclip.so")
    if native == "unreadable":
        (top / "_native.so").write_text("not a library")
    code = ("import paper_2108_01624_amd as pkg\n"
            "try:\n    pkg.load_library()\n"
            "except RuntimeError as e:\n    print('REFUSED', e, type(e.__cause__).__name__)\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=tmp_path, timeout=600, env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert "REFUSED" in r.stdout and "_native.so" in r.stdout and "python -m paper_2108_01624_amd.build" in r.stdout, r.stdout
    assert r.stdout.rstrip().endswith("ImportError" if native == "unreadable" else "NoneType")


@pytest.mark.parametrize("step", ["link of _native.so", "link"])
def test_a_build_that_fails_replaces_neither_file(monkeypatch, tmp_path, step):
    """A link that fails leaves the library and the extension of the last build, which fit one another."""
    from paper_2108_01624_amd import build

    for name in ("LIB_PATH", "NATIVE_PATH"):
        path = str(tmp_path / os.path.basename(getattr(build, name)))
        open(path, "w").write("old")
        monkeypatch.setattr(build, name, path)
    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path / "_build"))
    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build, "_compile_native", lambda: "native.o")

    def run(cmd, what):
        if what == step:
            raise RuntimeError(f"{what} failed")
        open(cmd[cmd.index("-o") + 1], "w").write("new")

    monkeypatch.setattr(build, "_run", run)
    with pytest.raises(RuntimeError, match="failed"):
        build.build_library()
    assert open(build.LIB_PATH).read() == open(build.NATIVE_PATH).read() == "old"
    step = "none"
    build.build_library()
    assert open(build.LIB_PATH).read() == open(build.NATIVE_PATH).read() == "new"

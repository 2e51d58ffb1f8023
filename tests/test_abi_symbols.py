"""The C-ABI library builds, loads and exports every symbol the header declares (no GPU needed)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mlora.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2605_13779_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2605_13779_amd import build
        build.build()
    return binding.load_library()


def declared_functions():
    text = re.sub(r"/\*.*?\*/", "", open(HEADER).read(), flags=re.S)
    names = re.findall(r"\b([a-z_0-9]+)\s*\(", text)
    return sorted({n for n in names if n.startswith(("mlora_", "lora_", "moe_"))})


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert {"lora_slots_upload", "lora_apply_decode", "lora_apply_segmented", "moe_lora_apply_packed"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_binding_covers_the_header():
    from paper_2605_13779_amd import binding
    assert set(declared_functions()) == set(binding.SIGNATURES)


def test_host_side_validation_without_a_gpu(lib):
    from paper_2605_13779_amd.binding import SiteDesc
    sz = [C.c_size_t() for _ in range(4)]
    ok = SiteDesc(2560, 9728, 16, 64, 0, 0)
    assert lib.mlora_site_bytes(C.byref(ok), *[C.byref(s) for s in sz]) == 0
    assert sz[0].value == 64 * 16 * 2560 * 2 and sz[1].value == 64 * 9728 * 16 * 2
    pad = SiteDesc(64, 64, 3, 2, 0, 0)      # r_max 3 is stored with stride 4
    assert lib.mlora_site_bytes(C.byref(pad), *[C.byref(s) for s in sz]) == 0
    assert sz[0].value == 2 * 4 * 64 * 2
    moe = SiteDesc(2048, 768, 8, 32, 128, 0)
    assert lib.mlora_site_bytes(C.byref(moe), *[C.byref(s) for s in sz]) == 0
    assert sz[0].value == 32 * 128 * 8 * 2048 * 2 and sz[1].value == 32 * 128 * 768 * 8 * 2
    for bad, code in [(SiteDesc(100, 64, 8, 2, 0, 0), -2), (SiteDesc(64, 64, 0, 2, 0, 0), -2),
                      (SiteDesc(64, 64, 65, 2, 0, 0), -2), (SiteDesc(64, 64, 8, 0, 0, 0), -1),
                      (SiteDesc(-8, 64, 8, 2, 0, 0), -1)]:
        assert lib.mlora_site_bytes(C.byref(bad), *[C.byref(s) for s in sz]) == code
    assert lib.mlora_site_bytes(None, *[C.byref(s) for s in sz]) == -1
    n = C.c_size_t()
    assert lib.mlora_plan_bytes(256, 64, C.byref(n)) == 0 and n.value % 256 == 0 and n.value > 256 * 16
    assert lib.mlora_plan_bytes(0, 64, C.byref(n)) == -1
    assert lib.mlora_status_str(-4) == b"segment offsets malformed"
    # null handles are rejected before any device work
    assert lib.lora_apply_decode(None, None, 0, None, 0, None, 4, None) == -1
    assert lib.lora_slots_upload(None, 0, 0, None, None, 1, 1.0, 0, None) == -1
    assert lib.moe_lora_apply_packed(None, None, 0, None, 0, None, None, 1, 1, None, None, None) == -1


def test_noop_is_rejected_by_the_parity_rules():
    """Mutation control for the comparison rules themselves: an implementation that leaves y
    unchanged must fail the delta check that every GPU parity test applies."""
    from tests import parity as P
    delta = np.random.default_rng(0).standard_normal((8, 16)) * 0.02
    with pytest.raises(AssertionError):
        P.noop_must_fail(np.zeros((8, 16), np.uint16), np.zeros((8, 16)), np.arange(8))
    P.noop_must_fail(np.zeros((8, 16), np.uint16), delta, np.arange(8))


def test_pack_experts_stacks_and_pads_like_numpy(lib):
    """Host-only packing of per-expert tensors into the slot image (the packed adapter form: one
    stacked tensor per projection and A|B instead of one per expert), against plain numpy."""
    from paper_2605_13779_amd import binding
    g = np.random.default_rng(7)
    for E, r, r_max, d_in, d_out in [(5, 3, 6, 24, 16), (4, 8, 8, 16, 40), (1, 1, 1, 8, 8), (128, 8, 8, 64, 24)]:
        desc = binding.SiteDesc(d_in, d_out, r_max, 2, E if E > 1 else 0, 0)
        A_e = [g.integers(1, 65535, size=(r, d_in), dtype=np.uint16) for _ in range(E)]
        B_e = [g.integers(1, 65535, size=(d_out, r), dtype=np.uint16) for _ in range(E)]
        a_img, b_img = binding.pack_experts(desc, A_e, B_e, r)
        rp = 1
        while rp < r_max:
            rp *= 2
        want_a = np.zeros((E, rp, d_in), dtype=np.uint16)
        want_b = np.zeros((E, d_out, rp), dtype=np.uint16)
        want_a[:, :r] = np.stack(A_e)
        want_b[:, :, :r] = np.stack(B_e)
        assert np.array_equal(a_img.reshape(E, rp, d_in), want_a)
        assert np.array_equal(b_img.reshape(E, d_out, rp), want_b)
    # the census of the paper's 30B-MoE adapter: per layer and projection 128 experts x {A, B} = 256
    # tensors become 2 stacked ones, 48 layers x 3 projections -> 36,864 become 288
    # (tests/golden/adapter_census.txt holds the printed totals)
    assert 48 * 3 * 128 * 2 == 36864 and 48 * 3 * 2 == 288
    desc = binding.SiteDesc(16, 16, 4, 2, 3, 0)
    A_e = [np.ones((2, 16), dtype=np.uint16)] * 3
    B_e = [np.ones((16, 2), dtype=np.uint16)] * 3
    with pytest.raises(binding.MLoraError):
        binding.pack_experts(desc, A_e, B_e, 5)        # rank above r_max


def test_switches_refuse_tile_heights_without_room(lib):
    """A plan has room for as many tile records as chunks, so tiles of fewer than four rows would be written past its
    end; the tile kernels take up to 16 rows."""
    for name in (b"tile_rows", b"tile_moe_rows"):
        for bad in (1, 2, 3, 17, 1 << 30):
            assert lib.mlora_set_tuning(name, bad) == -1, (name, bad)
        for good in (4, 16, -1, 0):
            assert lib.mlora_set_tuning(name, good) == 0, (name, good)
    assert lib.mlora_set_tuning(b"no such switch", 1) == -1


def test_earlier_name_of_a_switch(lib):
    assert lib.mlora_set_tuning(b"seg_no_mfma", 1) == 0
    assert lib.mlora_set_tuning(b"seg_no_mfma", 0) == 0


def test_wide_inline_stores_wait():
    """A store of more than 64 bits in inline assembly carries the two wait states its data registers need (the
    compiler adds them behind its own stores only; without them the first word of a store was overwritten now and
    then: prompts of 3130 rows, 9536 -> 9736 at rank 24, were 1.4 % off in norm)."""
    import glob
    here = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    found = 0
    for path in glob.glob(os.path.join(here, "paper_2605_13779_amd", "csrc", "*.h*")):
        with open(path) as f:
            for text in re.findall(r'asm volatile\("([^"]*store_dwordx[34][^"]*)"', f.read()):
                found += 1
                assert text.endswith("\\n\\ts_nop 1"), (path, text)
    assert found


def test_one_thread_reads_the_launch_tag():
    """A launch whose workgroups trade partial sums advances its tag as soon as every workgroup has signed in, and the
    sign-in is one thread's.  So that thread alone reads the tag, and the others take it from LDS behind a barrier: a
    wave that reads it by itself may see the next launch's."""
    here = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    text = {}
    for name in ("tile_multi.hip", "tile_body.h", "seg_mfma.hip"):
        with open(os.path.join(here, "paper_2605_13779_amd", "csrc", name)) as f:
            text[name] = re.sub(r"//[^\n]*", "", f.read())
    for name, reads in (("tile_multi.hip", 1), ("tile_body.h", 0), ("seg_mfma.hip", 1)):
        found = list(re.finditer(r"([\w.]+) = tag_read\(", text[name]))
        assert len(found) == reads, name
        for m in found:
            guard = text[name][:m.start()].rstrip()
            guard = guard[max(guard.rfind(";"), guard.rfind("}")):]                 # the statement the read belongs to
            assert re.search(r"\bthreadIdx\.x == 0\)", guard), (name, guard)
    for name, put, wait, take in (("tile_body.h", "s_tag = trade.tag;", "sums_to_lds();", "readfirstlane(s_tag)"),
                                  ("seg_mfma.hip", "s_epoch = e;", "__syncthreads();", "= s_epoch;")):
        at = text[name].index(put)
        assert "tid == 0" in text[name][at - 120:at] or "threadIdx.x == 0" in text[name][at - 120:at], name
        at = text[name].index(wait, at)
        assert take in text[name][at:] and take not in text[name][:at], name
    sums = text["tile_body.h"]
    sums = sums[sums.index("auto sums_to_lds ="):]
    assert "__syncthreads();" in sums[:sums.index("};")]


def test_down_form_for_few_tokens(lib):
    """The down projection's choice of form (host code): a decode step of few tokens always goes token by token up to rank
    16, and up to a token per CU the choice never flips back as tokens get fewer.  Large batches keep the two launches."""
    takes = lib._ZN5mlora21moe_down_takes_tokensEiiiiiiii
    takes.restype, takes.argtypes = C.c_bool, [C.c_int] * 8
    rng = np.random.default_rng(5)
    cus = 256
    for _ in range(300):
        E = int(rng.choice([1, 2, 4, 8, 16, 32, 64, 128, 200]))
        K, S, r = int(rng.integers(1, min(E, 16) + 1)), int(rng.integers(1, 65)), int(rng.choice([1, 2, 4, 8, 16]))
        d_in, d_out = 8 * int(rng.integers(1, 257)), 8 * int(rng.integers(1, 513))
        by_token = [takes(T, K, E, S, r, d_in, d_out, cus) for T in range(1, cus + 1)]
        assert all(by_token[:8]), (K, E, S, r, d_in, d_out)
        assert by_token == sorted(by_token, reverse=True), (K, E, S, r, d_in, d_out)
        assert not takes(100, K, E, S, 32, d_in, d_out, cus)
    for r in (8, 16):
        for T in (1, 2, 3, 4, 48, 100):
            assert takes(T, 8, 128, 32, r, 768, 2048, cus) and takes(T, 8, 128, 16, r, 1536, 4096, cus)
        assert not takes(2048, 8, 128, 32, r, 768, 2048, cus)
    assert takes(64, 4, 16, 8, 8, 1024, 4096, cus) and not takes(256, 4, 16, 8, 8, 1024, 4096, cus)

"""CPU-only checks of the C-ABI library: it loads without a GPU, exports every symbol the
header declares, and rejects bad arguments before touching a device."""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2602_17050_amd", "libmpzch.so")
HEADER = os.path.join(ROOT, "include", "mpzch.h")


@pytest.fixture(scope="module")
def binding():
    if not os.path.exists(LIB):
        from paper_2602_17050_amd import build
        build.build_library()
    from paper_2602_17050_amd import binding as b
    b.load_library()
    return b


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mpzch_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(binding):
    lib = ctypes.CDLL(LIB)
    names = declared_symbols()
    assert "mpzch_create" in names and "mpzch_remap" in names and "mpzch_lookup" in names
    assert "mpzch_reset_rows" in names and "mpzch_remap_jagged" in names
    for n in names:
        assert hasattr(lib, n), n
    assert set(binding.EXPORTED) == set(names)


def test_binding_uses_the_c_abi_names(binding):
    for n in binding.EXPORTED:
        assert callable(getattr(binding, n)), n


def test_create_validates_arguments_without_a_gpu(binding):
    b = binding
    h = b.mpzch_create(4096, 8, (b.EVICT_TTL, 3), 0x5EED)
    b.mpzch_destroy(h)
    h = b.mpzch_create(10, 64, (b.EVICT_NONE, 0), 1)        # max_probe > num_slots is accepted
    b.mpzch_destroy(h)
    for args in [(0, 8, (b.EVICT_TTL, 3)), (16, 0, (b.EVICT_TTL, 3)), (16, 8, (b.EVICT_TTL, -1)),
                 (16, 8, (7, 0)), (16, (1 << 20) + 1, (b.EVICT_NONE, 0))]:
        with pytest.raises(b.MpzchError) as e:
            b.mpzch_create(args[0], args[1], args[2], 0)
        assert e.value.status == 1
    b.mpzch_destroy(b.mpzch_create(16, 8, (b.EVICT_LRU, 0), 0))
    with pytest.raises(b.MpzchError) as e:
        b.mpzch_create(5000, 1025, (b.EVICT_LRU, 0), 0)      # LRU: max_probe <= 1024
    assert e.value.status == 4
    assert b.mpzch_status_string(0) == "ok"
    assert b.mpzch_status_string(1) == "invalid argument"


def test_entry_points_reject_bad_arguments_before_touching_the_gpu(binding):
    """Checks that run before the first HIP call: NULL handles and required pointers, sizes out of range, a slot
    count beyond MPZCH_MAX_SLOTS, a table that would reach past the 48 bits that a device address has."""
    b = binding
    lib = b.load_library()
    vp = ctypes.c_void_p
    h = b.mpzch_create(1000, 8, (b.EVICT_TTL, 1), 0)
    fake = vp(0x10000)                                        # never dereferenced: every call below fails first
    INVALID = 1
    assert lib.mpzch_remap(None, fake, fake, fake, 4, 1, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_remap(h, None, fake, fake, 4, 1, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_remap(h, fake, fake, fake, -1, 1, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_remap(h, fake, fake, fake, (1 << 30) + 1, 1, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_remap(h, fake, fake, fake, 4, -1, fake, fake, 4, fake, None, None) == INVALID      # step < 0
    assert lib.mpzch_remap(h, fake, fake, fake, 4, 1, None, fake, 4, fake, None, None) == INVALID       # no out_slots
    assert lib.mpzch_remap(h, fake, fake, fake, 4, 1, fake, None, 4, fake, None, None) == INVALID       # list of 4, no pointer
    high = vp((1 << 48) - 4096)                                # identities would end beyond 2^48
    assert lib.mpzch_remap(h, high, fake, fake, 4, 1, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_lookup(h, high, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_remap_reset(h, fake, fake, fake, 4, 1, fake, fake, 4, fake, None, None, 10, 16, 16, None, None) == INVALID
    assert lib.mpzch_remap_reset(h, fake, fake, fake, 4, 1, fake, fake, 4, fake, None, fake, 0, 16, 16, None, None) == INVALID
    assert lib.mpzch_remap_reset(h, fake, fake, fake, 4, 1, fake, fake, 4, fake, None, fake, 10, 6, 8, None, None) == INVALID
    assert lib.mpzch_remap_noalloc(h, fake, fake, fake, b.NOALLOC_MAX_BATCH + 1, 1, fake, fake, 4, fake, None, None) == 5
    assert lib.mpzch_lookup(None, fake, fake, 4, fake, None, None) == INVALID
    assert lib.mpzch_lookup_gather(h, fake, fake, 4, None, 10, 16, 16, fake, None, None, None) == INVALID  # no rows
    assert lib.mpzch_reset_rows(fake, fake, 4, fake, 10, 6, 8, None, None) == INVALID                       # 6-byte rows
    assert lib.mpzch_reserve(h, -1) == INVALID
    b.mpzch_destroy(h)
    with pytest.raises(b.MpzchError) as e:
        b.mpzch_create((1 << 40) + 1, 8, (b.EVICT_TTL, 1), 0)
    assert e.value.status == INVALID
    hr = b.mpzch_create_with_layout(1000, 8, (b.EVICT_TTL, 1), 0, b.LAYOUT_RECORDS)
    assert lib.mpzch_lookup(hr, vp(0x10008), fake, 4, fake, None, None) == INVALID      # records not 16-byte aligned
    assert lib.mpzch_remap(hr, vp(0x10000), vp(0x10004), fake, 4, 1, fake, fake, 4, fake, None, None) == INVALID  # metadata elsewhere
    b.mpzch_destroy(hr)
    with pytest.raises(b.MpzchError):
        b.mpzch_create_with_layout(1000, 8, (b.EVICT_TTL, 1), 0, 2)


def test_group_create_validates_arguments(binding):
    b = binding
    hs = [b.mpzch_create(100 + i, 4, (b.EVICT_TTL, 1), i) for i in range(3)]
    g = b.mpzch_group_create(hs)
    for h in hs:
        b.mpzch_destroy(h)                                   # the group keeps its own copy of the configs
    b.mpzch_group_destroy(g)
    with pytest.raises(b.MpzchError):
        b.mpzch_group_create([])
    h = b.mpzch_create(100, 4, (b.EVICT_LRU, 0), 0)
    b.mpzch_group_destroy(b.mpzch_group_create([h]))          # every policy may sit in a group
    b.mpzch_destroy(h)


def test_missing_library_fails_loudly(binding, tmp_path):
    with pytest.raises(FileNotFoundError):
        binding.load_library(str(tmp_path / "libmpzch.so"))


# A kernel's arguments are passed on as its parameters' types: a wrong pointer or a number that would lose bits must not
# compile (syntax only, host side)
@pytest.mark.parametrize("args,ok", [("(int32_t *)nullptr, (int64_t)5, (int32_t)7", True),
                                     ("(int32_t *)nullptr, (int64_t)5, (int64_t)7", False),
                                     ("(int64_t *)nullptr, (int64_t)5, (int32_t)7", False),
                                     ("(const int32_t *)nullptr, (int64_t)5, (int32_t)7", False)])
def test_launch_takes_only_arguments_that_fit(tmp_path, args, ok):
    from paper_2602_17050_amd import build
    src = tmp_path / "probe.hip"
    src.write_text('#include "mpzch.hip"\n'
                   f"static mpzch_status_t probe() {{ return launch(k_fill32, 1, 64, hipStream_t(nullptr), {args}); }}\n"
                   "void *probe_used = (void *)probe;\n")
    r = subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "--offload-host-only", "-fsyntax-only",
                        "-I", os.path.dirname(build.SRC), "-x", "hip", str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr[-2000:]


# The fields of an LRU claim tag are as wide as the limits of the header need: with a wider limit the library must not compile
# (syntax only, host side)
@pytest.mark.parametrize("limit,value,message", [("MPZCH_MAX_PROBE_LRU", "1024", ""), ("MPZCH_MAX_PROBE_LRU", "2049", "rounds"),
                                                 ("MPZCH_MAX_BATCH", "((int64_t)1 << 32) + 1", "positions")])
def test_lru_claim_tag_is_as_wide_as_the_limits(tmp_path, limit, value, message):
    from paper_2602_17050_amd import build
    src = tmp_path / "probe.hip"
    header = os.path.join(os.path.dirname(build.SRC), "..", "..", "include", "mpzch.h")
    src.write_text(f'#include "{header}"\n#undef {limit}\n#define {limit} ({value})\n#include "mpzch.hip"\n')
    r = subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "--offload-host-only", "-fsyntax-only",
                        "-I", os.path.dirname(build.SRC), "-x", "hip", str(src)], capture_output=True, text=True)
    if not message:
        assert r.returncode == 0, r.stderr[-2000:]
    else:
        assert r.returncode != 0 and any("static assertion" in x and message in x and "LRU claim tag" in x for x in r.stderr.splitlines()), r.stderr[-2000:]

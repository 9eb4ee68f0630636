"""Host-side checks that need no GPU: the C-ABI library loads, exports every symbol the
header declares, and its pure host helpers behave.  No kernel is launched here."""
import ctypes
import os
import re

import pytest

from paper_1905_03381_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_symbols():
    text = open(os.path.join(ROOT, "include", "autoassist.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(aa_[a-z0-9_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(api.LIB_PATH):
        from paper_1905_03381_amd import build
        build.build(force=False)
    return api.lib()


def test_library_exports_every_declared_symbol(L):
    names = header_symbols()
    assert len(names) >= 15
    for name in names:
        assert hasattr(L, name), f"{name} declared in the header but not exported"
    assert sorted(api.SYMBOLS) == names, "binding and header list different entry points"


def test_version_and_status_strings(L):
    assert api.version() >= 100
    seen = set()
    for code in (0, -1, -2, -3, -4, -5):
        s = api.status_string(code)
        assert s and s != "unknown status"
        seen.add(s)
    assert len(seen) == 6
    assert api.status_string(-99) == "unknown status"


def test_workspace_bytes_cover_every_use(L):
    small = api.workspace_bytes(256, 128)
    dense = api.workspace_bytes(16384, 1024)
    wide = api.workspace_bytes(16384, 2048)
    sparse = api.workspace_bytes(65536, 1 << 20)
    assert 0 < small <= dense <= wide
    # dense partials: up to 1024 blocks x 2 vectors x d floats
    assert dense >= 1024 * 2 * 1024 * 4 + 16384 * 5
    # CSR accumulators: 2 d floats; a later narrower dense call still fits
    assert sparse >= 2 * (1 << 20) * 4 + 65536 * 5
    assert sparse >= api.workspace_bytes(65536, 2048)
    assert api.workspace_bytes(-5, 0) > 0


def test_struct_layouts_match_the_header():
    assert ctypes.sizeof(api.aa_features) == 56
    assert api.aa_features.x.offset == 16 and api.aa_features.rowptr.offset == 32
    assert ctypes.sizeof(api.aa_step_config) == 48
    assert api.aa_step_config.seed.offset == 24 and api.aa_step_config.T.offset == 40


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(api, "_lib", None)
    monkeypatch.setattr(api, "LIB_PATH", "/nonexistent/libautoassist.so")
    with pytest.raises(api.AAError):
        api.lib()


def test_no_kernel_spills_registers():
    """The compiler's own report (written next to the objects by the build): no kernel of
    the library uses scratch memory.  A kernel that does parks values in memory one load at
    a time and its waves start late; on this target that has cost a factor of two."""
    from paper_1905_03381_amd import build
    try:
        table = build.kernel_resources()
    except FileNotFoundError:
        build.build(force=True)
        table = build.kernel_resources()
    assert len(table) > 50, "the resource remarks were not parsed"
    assert all("scratch" in v and "vgprs" in v for v in table.values())
    spilled = {k: v for k, v in table.items() if v["scratch"] > 0}
    assert not spilled, f"kernels with scratch: {spilled}"


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_stream_without_the_private_torch_calls(monkeypatch, missing):
    """A torch without the private pair is asked for its Stream object."""
    class Stream:
        cuda_stream = 1234

    monkeypatch.setattr(api, missing, None)
    monkeypatch.setattr(api.torch.cuda, "current_stream", lambda: Stream)
    assert api._stream() == 1234

"""What the benchmark reports about the profile kernels (no GPU): HBM traffic from
the committed measurement while the build's machine code is the one measured, and
the kernel that runs each length."""
import ctypes

import pytest

import bench
from paper_2401_13680_amd import _lib, api, build


@pytest.mark.parametrize("same", [True, False])
def test_traffic_of_the_measured_code(tmp_path, monkeypatch, same):
    note, built = tmp_path / "note.md", tmp_path / "sha"
    note.write_text("# traffic\n\n- profile kernels code sha256: `abc`\n- hbm bytes per cell: `3.5`\n")
    built.write_text("abc\n" if same else "abd\n")
    monkeypatch.setattr(bench, "TRAFFIC_NOTE", str(note))
    monkeypatch.setattr(bench, "KERNEL_HASH", str(built))
    assert bench.measured_traffic(2.0) == (7.0 if same else None)
    assert bench.measured_traffic(2.0, "another field") is None


def test_committed_note_is_of_the_hashed_kernels():
    fields = dict(line[2:].split(": ", 1) for line in open(bench.TRAFFIC_NOTE) if line.startswith("- ") and ": " in line)
    assert fields["kernels"].strip() == "k_stream, k_profile"
    assert len(fields["profile kernels code sha256"].strip(" `\n")) == 64
    for f in ("hbm bytes per cell", "hbm bytes per cell at m=256"):
        assert 0.5 < float(fields[f].strip(" `\n")) < 20


@pytest.mark.parametrize("m", [64, 128, 256, 512, 1024])
def test_kernel_reported_by_length(m):
    w = m - m // 2 + 1
    builtin = api.geometry(w)
    got = bench.profile_kernel(200_000, m, m // 2, builtin)
    assert got == dict(kernel="k_stream", windows_per_strip=992 if w <= 178 else 1984)
    other = next(c for c in api.geometry_candidates(w) if c != builtin)
    try:
        api.set_geometry(w, other)
        got = bench.profile_kernel(200_000, m, m // 2, builtin)
        assert got["kernel"] == "k_profile" and got["threads"] == api.decode_geometry(other)["threads"]
    finally:
        api.set_geometry(w, 0)

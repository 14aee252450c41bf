"""The build passes the compiler's warnings on; the host pass's message about the
device-only feature, several to a file, is left out."""
from paper_2503_12886_amd.csrc import build


def test_warnings():
    host = "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)\n"
    warning = "x.hip:3:1: warning: failed to meet occupancy target [-Wpass-failed]\n    3 | __global__\n"
    assert build.warnings(host * 3) == ""
    assert build.warnings(host + warning + host) == warning


def test_a_file_that_warns(tmp_path, capfd, monkeypatch):
    src = tmp_path / "w.hip"
    src.write_text("#warning seen\nint f() { return 0; }\n")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    build._compile("w.hip", str(tmp_path / "w.o"))
    err = capfd.readouterr().err
    assert "seen" in err and "packed-fp32-ops" not in err

"""compress_image where no further stream, or no pinned memory for one, is to be
had (CPU only, tests/host_image_streams.cpp): the channels then follow one
another on the context's own stream, as a context's first images do."""
from host_cc import run_host


def test_image_without_further_streams(tmp_path):
    run = run_host("host_image_streams.cpp", tmp_path)
    assert run.returncode == 0, run.stdout

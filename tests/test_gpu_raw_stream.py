"""The stream handle that the library's calls get is that of torch's current
stream, also where torch lacks the private functions that hand it out."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("missing", [None, "_raw_handle", "_raw_device"])
def test_raw_stream_is_the_current_stream(monkeypatch, missing):
    import torch
    from paper_2606_29794_amd import raster
    if missing:
        monkeypatch.setattr(raster, missing, None)
    dev = torch.device("cuda", torch.cuda.current_device())
    for s in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            for d in (None, torch.device("cuda"), dev):
                assert raster._raw_stream(d) == s.cuda_stream
            assert (raster._stream().value or 0) == s.cuda_stream

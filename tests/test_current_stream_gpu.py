"""The binding's default stream is torch's current stream: in the default case, inside
a stream context, in another thread and under graph capture."""
import threading

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["default", "context", "thread", "capture"])
def test_current_stream(where):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03325_amd import epb as E
    seen = []

    def look():
        seen.append((E._stream(None), torch.cuda.current_stream().cuda_stream))

    side = torch.cuda.Stream()
    if where == "default":
        look()
    elif where == "context":
        with torch.cuda.stream(side):
            look()
        assert seen[0][0] == side.cuda_stream
    elif where == "thread":
        with torch.cuda.stream(side):  # (the current stream is per thread)
            t = threading.Thread(target=look)
            t.start()
            t.join()
        assert seen[0][0] != side.cuda_stream
    else:
        x = torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=side):
            look()
            x.add_(1)
        assert seen[0][0] == side.cuda_stream
    assert seen and all(a == b for a, b in seen)

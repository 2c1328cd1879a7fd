"""The binding's per-call host path: the stream a call is put on is the
caller's current one, inside and outside a stream context, and what is no
contiguous GPU tensor of the stated type and shape is refused."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def test_current_stream():
    def handles():
        return llp._stream().value or 0, torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    seen = [handles()]
    with torch.cuda.stream(side):
        seen.append(handles())
    seen.append(handles())
    assert all(a == b for a, b in seen)
    assert seen[1][0] == side.cuda_stream != seen[0][0] == seen[2][0]


@pytest.mark.parametrize("bad", ["host", "dtype", "shape", "dims", "strided", "none", "list"])
def test_refused(bad):
    x = torch.zeros(6, 12, device="cuda")
    t = {"host": x.cpu(), "dtype": x.double(), "shape": x[:5], "dims": x[None],
         "strided": torch.zeros(12, 6, device="cuda").t(), "none": None, "list": x.tolist()}[bad]
    with pytest.raises(llp.LLPError) as e:
        llp._need(t, (6, 12), torch.float32, "x")
    assert e.value.status == llp.E_ARG
    llp._need(x, [6, 12], torch.float32, "x")

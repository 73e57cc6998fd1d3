"""4-D chunks of more than 2^30 values are counted in several launches: one
push of the whole image gives the curve of pushes of a few planes each (which
other tests compare with the oracle), the cuts within and between the pushes."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["u8", "u14", "u16"])
def test_cut_inside_a_push(dtype):
    import paper_1705_02045_amd as ecc
    shape = (4103, 64, 65, 63)
    print(f"\n[gpu] 4-D push of {shape} {dtype}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    bits = {"u8": 8, "u14": 14, "u16": 16}[dtype]
    kind = torch.uint8 if dtype == "u8" else torch.int16
    t = torch.empty(shape, dtype=kind, device="cuda")
    for i in range(0, shape[0], 512):  # (values of 16 bits as int16)
        part = t[i:i + 512]
        part.copy_(torch.randint(0, 1 << bits, part.shape, generator=g, device="cuda", dtype=torch.int32))
    curves = []
    for sizes in ([shape[0]], [4099, 4], [600] * 6 + [503]):
        st = ecc.Stream(shape, dtype)
        at = 0
        for n in sizes:
            st.push(t[at:at + n])
            at += n
        assert at == shape[0]
        curves.append(st.finish())
    assert int(curves[0][-1]) == 1
    assert (curves[0] == curves[2]).all() and (curves[1] == curves[2]).all()

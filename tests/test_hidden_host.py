"""The hidden-activation kernels without a GPU: which shapes they take, the workspace they ask for, and what they refuse
before touching HIP."""
from paper_2505_13813_amd import binding

STATUS = {"NULL": 1, "SHAPE": 2, "ALIGN": 4, "WORKSPACE": 5, "UNSUPPORTED": 8}


def test_supported_shapes():
    lib = binding.load_library()
    for K, N, G, yes in ((192, 768, 8, 1), (256, 1024, 8, 1), (384, 1536, 8, 1), (384, 384, 12, 1), (256, 256, 1, 1), (512, 2048, 8, 1), (640, 2560, 8, 1),
                         (192, 768, 32, 0),                       # d_g = 24
                         (384, 1024, 8, 0), (192, 200, 1, 0),     # no whole slabs
                         (192, 384 * 33, 1, 0),                   # more slabs than an XCD has compute units
                         (320, 1280, 8, 0), (768, 3072, 8, 1), (896, 3584, 8, 0), (384, 1536, 7, 0), (384, 1536, 0, 0), (0, 0, 0, 0)):
        assert lib.grkan_hidden_supported(K, N, G) == yes, (K, N, G)
        assert (lib.grkan_hidden_workspace_bytes(1000, K, N, G) > 0) == bool(yes)
    # [G][parts x wavefronts of a part in the group][10 sums]: 64 parts of 4 slabs, d_g = 192 in wavefronts of 32
    assert lib.grkan_hidden_workspace_bytes(25216, 384, 1536, 8) == 8 * 64 * 6 * 40
    assert lib.grkan_hidden_workspace_bytes(1, 384, 1536, 8) == 8 * 8 * 6 * 40
    assert lib.grkan_hidden_workspace_bytes(0, 384, 1536, 8) == 16
    assert lib.grkan_hidden_workspace_bytes(-1, 384, 1536, 8) == 0
    assert lib.grkan_hidden_workspace_bytes((1 << 30) + 1, 384, 1536, 8) == 0


def test_refusals():
    lib = binding.load_library()
    ok, p = 0, 1 << 20  # (an address that is never read)

    def fwd(y=p, W=p, bias=p, A=p, B=p, h=p, f=p, rows=64, K=384, N=1536, G=8):
        return lib.grkan_hidden_fwd(y, W, bias, A, B, h, f, rows, K, N, G, 1, None)

    def bwd(dout=p, W=p, h=p, A=p, B=p, dh=p, dA=p, dB=p, ws=p, bytes_=1 << 20, rows=64, K=384, N=1536, G=8):
        return lib.grkan_hidden_bwd(dout, W, h, A, B, dh, dA, dB, ws, bytes_, rows, K, N, G, 1, None)

    assert fwd(rows=0) == ok
    for call, status in ((fwd(rows=-1), "SHAPE"), (fwd(K=320, N=1280), "UNSUPPORTED"), (fwd(y=None), "NULL"), (fwd(h=None), "NULL"),
                         (fwd(y=p + 8), "ALIGN"), (fwd(bias=p + 2), "ALIGN"), (fwd(A=p + 1), "ALIGN"), (bwd(dA=None), "NULL"),
                         (bwd(dh=None), "NULL"), (bwd(h=p + 2), "ALIGN"), (bwd(ws=None), "WORKSPACE"), (bwd(bytes_=100), "WORKSPACE")):
        assert call == STATUS[status], (call, status)

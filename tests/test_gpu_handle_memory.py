"""Device memory of a cache handle (GPU only): a batch holds one handle per image, so what each takes besides its cache counts."""
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2410_01699_amd import synth  # noqa: E402

MIB = 1 << 20


def test_handle_of_7b_widths():
    """One layer of the 7B widths, 256 positions.  By the sizes in sjd_kv_create: cache 8 MiB, K-slices of the widest
    projection 43 (four outputs of 128 x 22016), FFN hidden 5.4, attention records 4.1, six [128 x 4096] matrices 12, rows
    of 256 logits 0.8: 74 MiB.  12 MiB more for the allocator's granularity (28 allocations)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_01699_amd import binding as B
    shape = synth.ModelShape(1, 4096, 32, 11008, 512, 256, 512, 256, synth.DTYPE_BF16)
    m = B.sjd_init_model(B.config_from_shape(shape), synth.make_weights(shape, seed=1, threads=16))
    kvs = [B.sjd_kv_create(m)]              # (the first also loads code)
    try:
        before = torch.cuda.mem_get_info()[0]
        kvs += [B.sjd_kv_create(m) for _ in range(4)]
        each = (before - torch.cuda.mem_get_info()[0]) / 4
        print(f"{each / MIB:.1f} MiB a handle", flush=True, file=sys.stderr)
        assert each < 86 * MIB
    finally:
        for kv in kvs:
            B.sjd_kv_free(kv)
        B.sjd_free_model(m)

"""Which kernel runs a bf16 product, on both sides of the lines of the dispatch: each was drawn where the one became the faster of the two.  The name of a
launch says the tile: 256 rows for the streamed products, none or 128 for the others.  (What they return: test_gpu_stream_products.py.)"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def rows(n, f):
    return torch.zeros(n, (f + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")[:, :f]


def launches(B, call):
    B.tma_profile_begin(None)
    call()
    return {name for name in B.tma_profile_end() if name.startswith("gemm_")}


def graph(n):
    return torch.zeros(n + 1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"), torch.ones(n, device="cuda")


def weights(fi, fo):
    return torch.zeros(fi, fo, device="cuda"), torch.zeros(fi, fo, device="cuda")


def forward(B, n, fi, fo):
    w = weights(fi, fo)
    Wt = B.tma_sage_prepare_weights_bf16(*w) if B.tma_sage_layer_aggregates_first(fi, fo, B.TMA_BF16) else None
    return launches(B, lambda: B.tma_sage_layer_fwd(*graph(n), rows(n, fi), *w, torch.zeros(fo, device="cuda"), B.TMA_ACT_NONE, Wt=Wt))


def test_rows_that_are_read_element_by_element_elsewhere(B):
    x = torch.zeros(65537, 102, dtype=torch.bfloat16, device="cuda")[:, :100]
    w = weights(100, 256)
    assert launches(B, lambda: B.tma_sage_layer_fwd(*graph(65537), x, *w, torch.zeros(256, device="cuda"), B.TMA_ACT_NONE,
                                                    Wt=B.tma_sage_prepare_weights_bf16(*w))) == {"gemm_fwd_256x256_bf16"}


def backward(B, n, fi, fo, relu, what):
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    got = launches(B, lambda: B.tma_sage_layer_bwd(*graph(n), rows(n, fi), rows(n, fi), rows(n, fo), rows(n, fo), *weights(fi, fo), act))
    return {name for name in got if what in name}


def dense(B, n, fi, fo, relu, what):
    act = B.TMA_ACT_RELU if relu else B.TMA_ACT_NONE
    got = launches(B, lambda: B.tma_dense_bwd(rows(n, fi), rows(n, fo), rows(n, fo), weights(fi, fo)[0], act))
    return {name for name in got if what in name}


@pytest.mark.parametrize("n,fi,fo,name", [(65536, 128, 256, "gemm_fwd_256x256_bf16"), (65536, 128, 260, "gemm_fwd_256x128_bf16"),
                                          (65536, 128, 384, "gemm_fwd_256x128_bf16"), (65536, 128, 385, "gemm_fwd_256x256_bf16"),
                                          (131071, 100, 300, "gemm_fwd_128x128_bf16"), (131072, 100, 300, "gemm_fwd_256x128_bf16"),
                                          (65536, 102, 300, "gemm_fwd_256x128_bf16"), (65536, 100, 256, "gemm_fwd_256x256_bf16"),
                                          (65537, 100, 256, "gemm_fwd_128x256_bf16"), (104704, 20, 256, "gemm_fwd_128x256_bf16"),
                                          (104705, 20, 256, "gemm_fwd_256x256_bf16"), (65537, 100, 200, "gemm_fwd_256x256_bf16"),
                                          (65537, 20, 200, "gemm_fwd_128x256_bf16"), (140000, 20, 200, "gemm_fwd_256x256_bf16"), (65537, 48, 256, "gemm_fwd_256x256_bf16"),
                                          (65536, 200, 300, "gemm_fwd_256x128_bf16"), (65536, 128, 301, "gemm_fwd_256x256_bf16"),
                                          (262143, 56, 300, "gemm_fwd_128x128_bf16"), (262144, 56, 300, "gemm_fwd_256x128_bf16"),
                                          (524287, 44, 400, "gemm_fwd_128x128_bf16"), (524288, 44, 400, "gemm_fwd_256x256_bf16"),
                                          (1048576, 20, 300, "gemm_fwd_128x128_bf16"), (1048576, 20, 400, "gemm_fwd_256x256_bf16")])
def test_forward(B, n, fi, fo, name):
    assert forward(B, n, fi, fo) == {name}


@pytest.mark.parametrize("n,fi,fo,relu,name", [(65536, 150, 128, False, "gemm_bwd_data_256x128_bf16"), (65536, 150, 128, True, "gemm_bwd_data_256x256_bf16"),
                                               (131071, 128, 100, False, "gemm_bwd_data_128x256_bf16"), (131072, 128, 100, False, "gemm_bwd_data_256x256_bf16"),
                                               (262143, 128, 100, True, "gemm_bwd_data_128x256_bf16"), (262144, 128, 100, True, "gemm_bwd_data_256x256_bf16"),
                                               (65536, 128, 102, True, "gemm_bwd_data_256x256_bf16"), (65536, 128, 132, True, "gemm_bwd_data_256x256_bf16"),
                                               (65536, 130, 100, False, "gemm_bwd_data_256x128_bf16"), (65536, 155, 128, False, "gemm_bwd_data_256x256_bf16"),
                                               (65536, 300, 160, False, "gemm_bwd_data_256x128_bf16")])
def test_input_gradient(B, n, fi, fo, relu, name):
    assert backward(B, n, fi, fo, relu, "bwd_data") == {name}


@pytest.mark.parametrize("n,fi,fo,relu,name", [(98304, 384, 256, False, "gemm_dense_bwd_data_256x128_bf16"),
                                               (98304, 384, 256, True, "gemm_dense_bwd_data_256x256_bf16"),
                                               (104704, 256, 100, False, "gemm_dense_bwd_data_bf16"), (104705, 256, 100, True, "gemm_dense_bwd_data_256x256_bf16"),
                                               (98304, 256, 132, True, "gemm_dense_bwd_data_256x256_bf16"), (524287, 384, 66, True, "gemm_dense_bwd_data_bf16"), (524288, 384, 66, True, "gemm_dense_bwd_data_256x256_bf16")])
def test_dense_input_gradient(B, n, fi, fo, relu, name):
    assert dense(B, n, fi, fo, relu, "bwd_data") == {name}


@pytest.mark.parametrize("n,fi,fo,name", [(98303, 256, 47, "gemm_tf_fwd_bf16"), (98304, 256, 47, "gemm_tf_fwd_256x96_bf16"),
                                          (131071, 128, 47, "gemm_tf_fwd_bf16"), (131072, 128, 47, "gemm_tf_fwd_256x96_bf16"),
                                          (131071, 256, 20, "gemm_tf_fwd_bf16"), (131072, 256, 20, "gemm_tf_fwd_256x96_bf16"),
                                          (524287, 128, 32, "gemm_tf_fwd_bf16"), (524288, 128, 32, "gemm_tf_fwd_256x96_bf16")])
def test_transform_first_forward(B, n, fi, fo, name):
    assert forward(B, n, fi, fo) == {name}


@pytest.mark.parametrize("n,fi,fo,name", [(131071, 256, 47, "gemm_tf_bwd_data_bf16"), (131072, 256, 47, "gemm_tf_bwd_data_256x256_bf16"),
                                          (262143, 128, 47, "gemm_tf_bwd_data_bf16"), (262144, 128, 47, "gemm_tf_bwd_data_256x128_bf16"),
                                          (262143, 256, 40, "gemm_tf_bwd_data_bf16"), (262144, 256, 40, "gemm_tf_bwd_data_256x256_bf16"),
                                          (1048575, 128, 40, "gemm_tf_bwd_data_bf16"), (1048576, 128, 40, "gemm_tf_bwd_data_256x128_bf16")])
def test_transform_first_input_gradient(B, n, fi, fo, name):
    assert backward(B, n, fi, fo, False, "bwd_data") == {name}


@pytest.mark.parametrize("n,fi,fo,relu,name", [(1048575, 64, 96, True, "gemm_bwd_weight_256x128_bf16"), (1048576, 64, 96, True, "gemm_bwd_weight_128x128_bf16"),
                                               (1048576, 64, 96, False, "gemm_bwd_weight_256x128_bf16"), (1048576, 72, 96, True, "gemm_bwd_weight_256x128_bf16"),
                                               (1048576, 64, 136, True, "gemm_bwd_weight_256x256_bf16"),
                                               (1048576, 128, 47, False, "gemm_tf_bwd_weight_256x128_bf16"), (1048576, 128, 20, False, "gemm_tf_bwd_weight_bf16"),
                                               (2097152, 64, 20, False, "gemm_tf_bwd_weight_256x128_bf16")])
def test_weight_gradient(B, n, fi, fo, relu, name):
    assert backward(B, n, fi, fo, relu, "bwd_weight") == {name}


@pytest.mark.parametrize("n,fi,fo,relu,name", [(98303, 256, 64, False, "gemm_dense_bwd_weight_bf16"), (98304, 256, 64, False, "gemm_dense_bwd_weight_256x128_bf16"),
                                               (131071, 256, 64, True, "gemm_dense_bwd_weight_bf16"), (131072, 256, 64, True, "gemm_dense_bwd_weight_256x128_bf16"),
                                               (65536, 512, 64, True, "gemm_dense_bwd_weight_256x128_bf16"),
                                               (2000000, 64, 96, True, "gemm_dense_bwd_weight_bf16"), (1048576, 64, 97, True, "gemm_dense_bwd_weight_256x128_bf16"),
                                               (1310719, 128, 64, False, "gemm_dense_bwd_weight_bf16"), (1310720, 128, 64, False, "gemm_dense_bwd_weight_256x128_bf16")])
def test_dense_weight_gradient(B, n, fi, fo, relu, name):
    assert dense(B, n, fi, fo, relu, "bwd_weight") == {name}


def test_narrowed_weights(B):
    """A launch's name stands for one kernel: bench.py refuses to match counters with launches otherwise."""
    def names(call):
        B.tma_profile_begin(None)
        call()
        return {name for name in B.tma_profile_end() if name.startswith(("narrow", "prepare"))}

    n, agg, tf = 131072, weights(128, 256), weights(256, 47)
    both = names(lambda: B.tma_sage_prepare_weights_bf16(*agg)) | names(
        lambda: B.tma_sage_layer_bwd(*graph(n), rows(n, 128), rows(n, 128), rows(n, 256), rows(n, 256), *agg, B.TMA_ACT_NONE))
    assert both == {"prepare_weights_bf16", "narrow_stack_bf16"}
    assert names(lambda: B.tma_sage_layer_fwd(*graph(n), rows(n, 256), *tf, torch.zeros(47, device="cuda"), B.TMA_ACT_NONE)) == {"narrow_sides_t_bf16"}
    assert names(lambda: B.tma_sage_layer_bwd(*graph(n), rows(n, 256), rows(n, 256), rows(n, 47), rows(n, 47), *tf, B.TMA_ACT_NONE)) == {"narrow_sides_bf16"}

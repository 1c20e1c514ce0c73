"""Calls that the fused launch of 5 to 16 tokens (two matrices: from 2 on) takes, beside the kernel it takes for them: units that a
wavefront keeps in flight, pieces of the quantizer that it holds (test_launches.py asks the library, test_gpu_stream_fused.py runs them).
Rows of one unit of 256 channels to seven a wavefront, in one task and in several across the ring's rounds; slices of K that stay empty or
end early; wavefronts that share a slice; one row group to more tasks than a workgroup keeps open."""

# (units, pieces), tokens, channels in, channels out
ONE = [((2, 8), 5, 256, 16), ((2, 8), 16, 768, 272), ((2, 8), 7, 1280, 528), ((2, 8), 6, 2048, 1040), ((2, 8), 9, 2304, 48),
       ((2, 8), 16, 4096, 4096), ((4, 8), 13, 4096, 14336), ((2, 8), 5, 8192, 4096), ((4, 8), 5, 8192, 8208), ((4, 8), 5, 6144, 12304),
       ((4, 8), 7, 4608, 16400), ((4, 8), 11, 1024, 66128), ((4, 8), 15, 512, 40000), ((2, 8), 8, 2048, 2048)]
# (units, pieces), tokens, channels in, channels out of the two matrices
TWO = [((4, 8), 2, 28672, 272, 16), ((4, 8), 2, 28672, 4112, 4096), ((4, 8), 3, 12288, 1040, 2064), ((4, 8), 3, 12288, 14336, 14336),
       ((2, 8), 5, 1024, 528, 272), ((2, 8), 12, 2048, 4096, 4096), ((4, 8), 16, 4096, 11008, 11008), ((2, 16), 16, 8192, 1008, 528),
       ((4, 16), 16, 8192, 11008, 11024), ((4, 16), 9, 8192, 4112, 8208), ((4, 16), 7, 15872, 2064, 3088), ((4, 8), 6, 256, 16, 33024),
       ((4, 16), 2, 65536, 272, 1040)]

// Host side of the index-time training entry points (included by ivf_gp.hip, after its helpers).
#pragma once

extern "C" int ivf_group(const int32_t *bucket, int64_t n, int64_t nbuckets, int32_t *perm, uint32_t *offsets,
                         void *hip_stream)
{
    if (!bucket || !perm || !offsets) return fail(IVF_EINVAL, "NULL argument");
    if (n < 0 || n >= (1ll << 32) - 1) return fail(IVF_EINVAL, "n=%lld out of range", (long long)n);
    if (nbuckets < 1 || nbuckets >= (1ll << 31)) return fail(IVF_EINVAL, "nbuckets=%lld out of range", (long long)nbuckets);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    RadixBufs rb;
    int rc = rb.init(n);
    if (!rc && n > 0) {
        auto body = [&]() -> int {
            HIPCHK(hipMemcpyAsync(rb.keys_a(), bucket, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
            uint32_t *ks, *vs;
            int r2 = rb.sort(n, bits_for(nbuckets), false, &ks, &vs, st);
            if (r2) return r2;
            bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, nbuckets, offsets);
            LAUNCHCHK("bucket_offsets_kernel");
            HIPCHK(hipMemcpyAsync(perm, vs, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
            return IVF_OK;
        };
        rc = body();
    } else if (!rc) {
        rc = hipMemsetAsync(offsets, 0, (size_t)(nbuckets + 1) * sizeof(uint32_t), st) == hipSuccess
                 ? IVF_OK : fail(IVF_EHIP, "hipMemsetAsync failed");
    }
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_gather_rows(const void *src, int64_t row_bytes, const int32_t *perm, int64_t n, void *dst,
                               void *hip_stream)
{
    if (!src || !perm || !dst) return fail(IVF_EINVAL, "NULL argument");
    if (row_bytes < 1 || n < 0) return fail(IVF_EINVAL, "bad sizes");
    if (n == 0) return IVF_OK;
    const uintptr_t al = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst) | (uintptr_t)row_bytes;
    const int vec = (al % 16 == 0) ? 16 : (al % 8 == 0) ? 8 : (al % 4 == 0) ? 4 : 1;
    const int64_t threads = n * (row_bytes / vec);
    if (threads >= (1ll << 32) - 256) return fail(IVF_EINVAL, "too many rows for one launch");
    gather_rows_kernel<<<dim3(grid_for(threads)), dim3(256), 0, static_cast<hipStream_t>(hip_stream)>>>(
        static_cast<const uint8_t *>(src), row_bytes, perm, n, static_cast<uint8_t *>(dst), vec);
    LAUNCHCHK("gather_rows_kernel");
    return IVF_OK;
}

extern "C" int ivf_bucket_ids(const int32_t *region, const int32_t *sub, int64_t n, int L, int32_t *bucket,
                              void *hip_stream)
{
    if (!region || !sub || !bucket) return fail(IVF_EINVAL, "NULL argument");
    if (n < 0 || L < 1) return fail(IVF_EINVAL, "bad sizes");
    if (n == 0) return IVF_OK;
    bucket_ids_kernel<<<dim3(grid_for(n)), dim3(256), 0, static_cast<hipStream_t>(hip_stream)>>>(region, sub, n, L, bucket);
    LAUNCHCHK("bucket_ids_kernel");
    return IVF_OK;
}

namespace {

// centroids[j] = mean of the rows perm[off[j]] .. of x
int launch_cluster_means(const float *x, int D, const uint32_t *perm, const uint32_t *off, int64_t K, float *centroids, hipStream_t st)
{
    const unsigned columns = (unsigned)((D + WAVE - 1) / WAVE);
    long_segment_mean_kernel<<<dim3((unsigned)(K < 256 ? K : 256), columns), dim3(1024), 0, st>>>(x, D, perm, off, K, centroids);
    LAUNCHCHK("long_segment_mean_kernel");
    if (D % 2 == 0) short_segment_mean_kernel<2><<<dim3(grid_for(K, 4), (columns + 1) / 2), dim3(256), 0, st>>>(x, D, perm, off, K, centroids);
    else short_segment_mean_kernel<1><<<dim3(grid_for(K, 4), columns), dim3(256), 0, st>>>(x, D, perm, off, K, centroids);
    LAUNCHCHK("short_segment_mean_kernel");
    return IVF_OK;
}

}  // namespace

extern "C" int ivf_cluster_means(const float *x, int64_t n, int D, const int32_t *assign, int64_t K,
                                 float *centroids, void *hip_stream)
{
    if (!x || !assign || !centroids) return fail(IVF_EINVAL, "NULL argument");
    if (D < 1 || D > IVF_MAX_D || K < 1 || K >= (1ll << 31)) return fail(IVF_EINVAL, "bad sizes");
    if (n < 0 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n out of range");
    if (n == 0) return IVF_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    RadixBufs rb;
    DevTmp off;
    auto body = [&]() -> int {
        int r2;
        if ((r2 = rb.init(n))) return r2;
        HIPCHK(off.alloc((size_t)(K + 1) * sizeof(uint32_t)));
        HIPCHK(hipMemcpyAsync(rb.keys_a(), assign, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
        uint32_t *ks, *vs;
        if ((r2 = rb.sort(n, bits_for(K), false, &ks, &vs, st))) return r2;
        bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, K, static_cast<uint32_t *>(off.p));
        LAUNCHCHK("bucket_offsets_kernel");
        if ((r2 = launch_cluster_means(x, D, vs, static_cast<uint32_t *>(off.p), K, centroids, st))) return r2;
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    int rc = body();
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_kmeans(const float *x, int64_t n, int D, int64_t K, int iters, const int64_t *init_idx,
                          float *centroids, double *objective, void *hip_stream)
{
    int rc = IVF_OK;
    if (!x || !init_idx || !centroids) return fail(IVF_EINVAL, "NULL argument");
    if (D < 4 || D % 4 || D > IVF_MAX_D) return fail(IVF_EINVAL, "D=%d must be a multiple of 4 in [4, %d]", D, IVF_MAX_D);
    if (n < 1 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n=%lld out of range", (long long)n);
    if (!aligned16(x)) return fail(IVF_EINVAL, "x must be 16-byte aligned");
    if (K < 1 || K > n) return fail(IVF_EINVAL, "need 1 <= K <= n");
    if (iters < 0) return fail(IVF_EINVAL, "iters must be >= 0");
    if (!aligned16(centroids)) return fail(IVF_EINVAL, "centroids must be 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ArgminCtx ctx;
    RadixBufs rb;
    DevTmp lab, dist, off;
    auto body = [&]() -> int {
        int r2;
        take_rows_kernel<<<dim3(grid_for(K * D)), dim3(256), 0, st>>>(x, D, 0, D, init_idx, K, centroids, D, 0);
        LAUNCHCHK("take_rows_kernel");
        if (iters == 0) return IVF_OK;
        if ((r2 = ctx.init(K, D, n, iters > 1))) return r2;
        if ((r2 = rb.init(n))) return r2;
        HIPCHK(lab.alloc((size_t)n * sizeof(int32_t)));
        if (objective) HIPCHK(dist.alloc((size_t)n * sizeof(float)));
        HIPCHK(off.alloc((size_t)(K + 1) * sizeof(uint32_t)));
        const int bits = bits_for(K);
        for (int it = 0; it < iters; ++it) {
            if ((r2 = ctx.set_centroids(centroids, st))) return r2;
            int32_t *lb = static_cast<int32_t *>(lab.p);
            if ((r2 = ctx.run(x, n, lb, objective ? static_cast<float *>(dist.p) : nullptr, st, -1, it ? lb : nullptr))) return r2;
            if (objective) {
                fixed_sum_kernel<float><<<dim3(1), dim3(1024), 0, st>>>(static_cast<float *>(dist.p), n, objective + it);
                LAUNCHCHK("fixed_sum_kernel");
            }
            HIPCHK(hipMemcpyAsync(rb.keys_a(), lab.p, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
            uint32_t *ks, *vs;
            if ((r2 = rb.sort(n, bits, false, &ks, &vs, st))) return r2;
            bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, K, static_cast<uint32_t *>(off.p));
            LAUNCHCHK("bucket_offsets_kernel");
            if ((r2 = launch_cluster_means(x, D, vs, static_cast<uint32_t *>(off.p), K, centroids, st))) return r2;
        }
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    rc = body();
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_pq_train(const float *E, int64_t n, int D, int M, int iters, const int64_t *init_idx,
                            float *codebook, void *hip_stream)
{
    if (!E || !init_idx || !codebook) return fail(IVF_EINVAL, "NULL argument");
    if (M < 1 || D < M || D % M || D > IVF_MAX_D) return fail(IVF_EINVAL, "D=%d must be a multiple of M=%d", D, M);
    if (n < 256 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n=%lld: need at least 256 training rows", (long long)n);
    if (iters < 0) return fail(IVF_EINVAL, "iters must be >= 0");
    const int ds = D / M;
    if (!pq_width(ds))
        return fail(IVF_EINVAL, "D/M=%d: the codeword assignment kernel is built for block widths 4, 6, 8, 12 and 16", ds);
    const size_t cb_bytes = (size_t)256 * D * sizeof(float);
    if (cb_bytes > 140 * 1024) return fail(IVF_EINVAL, "codebook of %zu bytes does not fit LDS", cb_bytes);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    RadixBufs rb;
    DevTmp codes, off, state, psum, pcnt;
    uint32_t seen[2];                            // largest magnitude, flag
    // all rounds, the means from fixed-point sums (exact unless the flag is raised) or from fp64 segment sums
    auto rounds = [&](bool fixed) -> int {
        int r2;
        uint8_t *cd = static_cast<uint8_t *>(codes.p);
        uint32_t *sw = static_cast<uint32_t *>(state.p);
        for (int m = 0; m < M; ++m) {   // codeword j of block m starts as block m of row init_idx[j]
            take_rows_kernel<<<dim3(grid_for(256 * ds)), dim3(256), 0, st>>>(E, D, m * ds, ds, init_idx, 256,
                                                                              codebook + (size_t)m * 256 * ds, ds, 0);
            LAUNCHCHK("take_rows_kernel");
        }
        for (int it = 0; it < iters; ++it) {
            // nearest codeword of every block of every row, by (distance, index)
            if ((r2 = launch_pq_encode(ds, E, nullptr, n, M, codebook, nullptr, cd, nullptr, nullptr, st))) return r2;
            // every codeword becomes the mean of the rows assigned to it
            if (fixed && (r2 = launch_pq_means(ds, E, n, M, cd, sw, static_cast<double *>(psum.p), static_cast<uint32_t *>(pcnt.p), codebook, st))) return r2;
            for (int m = 0; !fixed && m < M; ++m) {
                byte_column_kernel<<<dim3(grid_for(n)), dim3(256), 0, st>>>(cd, n, M, m, rb.keys_a());
                LAUNCHCHK("byte_column_kernel");
                uint32_t *ks, *vs;
                if ((r2 = rb.sort(n, 8, false, &ks, &vs, st))) return r2;
                bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, 256, static_cast<uint32_t *>(off.p));
                LAUNCHCHK("bucket_offsets_kernel");
                segment_sum_kernel<float, 1><<<dim3(256), dim3(256), 0, st>>>(
                    E, D, m * ds, ds, vs, static_cast<uint32_t *>(off.p), nullptr, codebook + (size_t)m * 256 * ds, ds, 0);
                LAUNCHCHK("segment_sum_kernel");
            }
        }
        if (iters) HIPCHK(hipMemcpyAsync(seen, state.p, sizeof(seen), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    auto body = [&]() -> int {
        if (iters == 0) return rounds(true);
        int r2;
        const size_t state_words = 2 + 2 * (size_t)M * 256 * (1 + ds), words = (size_t)pq_sum_slices(n) * M * 256;
        HIPCHK(codes.alloc((size_t)n * M));
        HIPCHK(state.alloc(state_words * sizeof(uint32_t)));
        HIPCHK(psum.alloc(words * ds * sizeof(double)));
        HIPCHK(pcnt.alloc(words * sizeof(uint32_t)));
        fill_u64_kernel<<<dim3(grid_for(state_words / 2)), dim3(256), 0, st>>>(static_cast<unsigned long long *>(state.p), state_words / 2, 0ull);
        LAUNCHCHK("fill_u64_kernel");
        if ((r2 = launch_absmax<false>(E, n * D, static_cast<uint32_t *>(state.p), st))) return r2;
        if ((r2 = rounds(true))) return r2;
        // (infinities and values that are not numbers have to find their way into the means: by the segment sums too)
        if (seen[0] < 0x7F800000u && !seen[1]) return IVF_OK;
        if ((r2 = rb.init(n))) return r2;
        HIPCHK(off.alloc(257 * sizeof(uint32_t)));
        return rounds(false);
    };
    int rc = body();
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_lloyd_1d(const float *t, int64_t n, int iters, float *table, void *hip_stream)
{
    if (!t || !table) return fail(IVF_EINVAL, "NULL argument");
    if (n < 1 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n out of range");
    if (iters < 0) return fail(IVF_EINVAL, "iters must be >= 0");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    RadixBufs rb;
    DevTmp sorted, off, sum;
    auto body = [&]() -> int {
        int r2;
        if ((r2 = rb.init(n))) return r2;
        HIPCHK(sorted.alloc((size_t)n * sizeof(float)));
        HIPCHK(off.alloc(257 * sizeof(uint32_t)));
        HIPCHK(sum.alloc(256 * sizeof(double)));
        float *s = static_cast<float *>(sorted.p);
        float_keys_kernel<<<dim3(grid_for(n)), dim3(256), 0, st>>>(t, n, rb.keys_a());
        LAUNCHCHK("float_keys_kernel");
        uint32_t *ks, *vs;
        if ((r2 = rb.sort(n, 32, false, &ks, &vs, st))) return r2;
        key_floats_kernel<<<dim3(grid_for(n)), dim3(256), 0, st>>>(ks, n, s);
        LAUNCHCHK("key_floats_kernel");
        lloyd1d_init_kernel<<<dim3(1), dim3(256), 0, st>>>(s, n, table);
        LAUNCHCHK("lloyd1d_init_kernel");
        int64_t grid = (n + 255) / 256;
        if (grid > 4096) grid = 4096;
        for (int it = 0; it < iters; ++it) {
            lloyd1d_label_kernel<<<dim3((unsigned)grid), dim3(256), 0, st>>>(s, n, table, rb.keys_a());
            LAUNCHCHK("lloyd1d_label_kernel");
            if ((r2 = rb.sort(n, 8, false, &ks, &vs, st))) return r2;
            bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, 256, static_cast<uint32_t *>(off.p));
            LAUNCHCHK("bucket_offsets_kernel");
            segment_sum_kernel<float, 0><<<dim3(256), dim3(256), 0, st>>>(s, 1, 0, 1, vs, static_cast<uint32_t *>(off.p),
                                                                          static_cast<double *>(sum.p), nullptr, 0, 0);
            LAUNCHCHK("segment_sum_kernel");
            lloyd1d_update_kernel<<<dim3(1), dim3(256), 0, st>>>(static_cast<double *>(sum.p), static_cast<uint32_t *>(off.p), table);
            LAUNCHCHK("lloyd1d_update_kernel");
        }
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    int rc = body();
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_learn_alpha(const float *centroids, int64_t K, int D, const int32_t *nbr, int L, const float *x,
                               int64_t n, const int32_t *region, float *alpha, void *hip_stream)
{
    if (!centroids || !nbr || !x || !region || !alpha) return fail(IVF_EINVAL, "NULL argument");
    if (D < 1 || D > IVF_MAX_D || K < 1 || K >= (1ll << 31) || L < 1) return fail(IVF_EINVAL, "bad sizes");
    if (n < 0 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n out of range");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    RadixBufs rb;
    DevTmp stat, off, nd, tot;
    auto body = [&]() -> int {
        int r2;
        if ((r2 = rb.init(n))) return r2;
        HIPCHK(stat.alloc((size_t)(n > 0 ? n : 1) * 2 * sizeof(double)));
        HIPCHK(off.alloc((size_t)(K + 1) * sizeof(uint32_t)));
        HIPCHK(nd.alloc((size_t)K * 2 * sizeof(double)));
        HIPCHK(tot.alloc(2 * sizeof(double)));
        HIPCHK(hipMemsetAsync(stat.p, 0, (size_t)(n > 0 ? n : 1) * 2 * sizeof(double), st));
        HIPCHK(hipMemsetAsync(off.p, 0, (size_t)(K + 1) * sizeof(uint32_t), st));
        if (n > 0) {
            alpha_point_kernel<<<dim3((unsigned)n), dim3(64), (size_t)D * sizeof(float), st>>>(
                x, n, D, L, region, centroids, nbr, static_cast<double *>(stat.p));
            LAUNCHCHK("alpha_point_kernel");
            HIPCHK(hipMemcpyAsync(rb.keys_a(), region, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
            uint32_t *ks, *vs;
            if ((r2 = rb.sort(n, bits_for(K), false, &ks, &vs, st))) return r2;
            bucket_offsets_kernel<<<dim3(grid_for(n + 1)), dim3(256), 0, st>>>(ks, n, K, static_cast<uint32_t *>(off.p));
            LAUNCHCHK("bucket_offsets_kernel");
            segment_sum_kernel<double, 0><<<dim3((unsigned)K), dim3(256), 0, st>>>(
                static_cast<double *>(stat.p), 2, 0, 2, vs, static_cast<uint32_t *>(off.p), static_cast<double *>(nd.p), nullptr, 0, 0);
            LAUNCHCHK("segment_sum_kernel");
        } else {
            HIPCHK(hipMemsetAsync(nd.p, 0, (size_t)K * 2 * sizeof(double), st));
        }
        // pooled ratio: the two sums over all regions, each in a fixed order (stride-2 views of nd)
        strided_sum_kernel<<<dim3(2), dim3(1024), 0, st>>>(static_cast<double *>(nd.p), K, 2, static_cast<double *>(tot.p));
        LAUNCHCHK("strided_sum_kernel");
        alpha_finish_kernel<<<dim3(grid_for(K)), dim3(256), 0, st>>>(static_cast<double *>(nd.p), static_cast<double *>(tot.p), K, alpha);
        LAUNCHCHK("alpha_finish_kernel");
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    int rc = body();
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_neighbours(const float *centroids, int64_t K, int D, int L, int32_t *nbr, float *cs_dist2,
                              void *hip_stream)
{
    int rc = check_coarse_args(centroids, K, D, centroids, K);
    if (rc) return rc;
    if (!nbr || !cs_dist2) return fail(IVF_EINVAL, "NULL argument");
    if (L < 1 || L >= K || L + 1 > 4096) return fail(IVF_EINVAL, "need 1 <= L < K and L <= 4095");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int P = L + 1;
    DevTmp tid, td;
    HIPCHK(tid.alloc((size_t)K * P * sizeof(int32_t)));
    HIPCHK(td.alloc((size_t)K * P * sizeof(float)));
    rc = coarse_topk_tiled(centroids, K, D, centroids, K, P, static_cast<int32_t *>(tid.p), static_cast<float *>(td.p), st);
    if (!rc) {
        neighbour_rows_kernel<<<dim3((unsigned)K), dim3(64), (size_t)P * sizeof(unsigned long long), st>>>(
            static_cast<int32_t *>(tid.p), static_cast<float *>(td.p), K, P, nbr, cs_dist2);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) rc = fail(IVF_EHIP, "launch neighbour_rows_kernel: %s", hipGetErrorString(e));
    }
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

// Batched refactorization: several bound handles (same device, same factor precision; the
// same or different patterns) refactored by one launch per dependency level across the
// whole batch, the value update merged likewise, and every launch of a batch step recorded
// once into a HIP graph that later steps replay.  Included by kkt_runtime.hip (it needs the
// handle's internals).
//
// Each launch is cut into shares, one per handle: share p runs blocks [blk0, blk0 + nblk)
// of the launch with that handle's arguments, so every handle's result is bitwise the same as
// refactoring it alone.  The refinement solves all handles' first systems in one launch per
// triangle, on tickets over an order of their items level by level, and reads all their norms
// back together; FGMRES follows handle by handle for those short of the target.

namespace kkt {

// Everything the batched kernels read of one handle.
template <class T>
struct BatchSys {
    RefArgs<T> ref;
    const int32_t *a_rowptr, *a_colind, *colptr, *Q;
    const int2 *lu_src;
    double *r, *c;
    int16_t *er, *ec;
    int n, eq, nb_norm;
    CopyRanges rest;   // the copy after the last level
    // refinement: the two triangles' solves (solutions and right-hand sides come with the call)
    SolveArgs<T> l, u;
    const int32_t *P;
    double *rpart;     // block maxima of the residual
};

// What the refinement of one handle reads back: its status block and residual norms.
struct BatchResult {
    DevStatus st;
    ResNorms rn;
};

// The call's pointers of one handle.
struct BatchPtrs {
    const double *v, *b;
    double *x;
};

// One handle's share of a batched launch.
struct BatchPart {
    int sys, blk0, nblk, item0, nwide, small0, nsmall;
    CopyRanges c;   // the level's chunk of the row-ordered copy
    int pad0;
};

// the share that runs block b (shares are sorted by blk0, the first starts at 0)
__device__ __forceinline__ int find_part(const BatchPart *__restrict__ parts, int nparts, int b) {
    int lo = 0, hi = nparts - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (parts[mid].blk0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_clear(const BatchSys<T> *__restrict__ sys) {
    clear_status_body(sys[blockIdx.x].ref.st, sys[blockIdx.x].ref.pcount);
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_rows(const BatchSys<T> *__restrict__ sys,
                                                    const BatchPart *__restrict__ parts, int nparts,
                                                    const double *const *__restrict__ vals) {
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const BatchSys<T> &S = sys[P.sys];
    row_scale_body(blockIdx.x - P.blk0, S.n, S.a_rowptr, vals[P.sys], S.eq, S.r, S.er, S.ref.st);
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_cols(const BatchSys<T> *__restrict__ sys,
                                                    const BatchPart *__restrict__ parts, int nparts,
                                                    const double *const *__restrict__ vals) {
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const BatchSys<T> &S = sys[P.sys];
    col_store_body<T>(blockIdx.x - P.blk0, S.n, S.colptr, S.lu_src, S.Q, vals[P.sys], S.er, S.eq, S.c, S.ec,
                      S.ref.lu);
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_rowsums(const BatchSys<T> *__restrict__ sys,
                                                       const BatchPart *__restrict__ parts, int nparts,
                                                       const double *const *__restrict__ vals) {
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const BatchSys<T> &S = sys[P.sys];
    norms_body(blockIdx.x - P.blk0, S.n, S.a_rowptr, S.a_colind, vals[P.sys], S.r, S.ec, S.ref.st);
}

template <class C>
__global__ __launch_bounds__(C::kThreads, C::kWaves) void k_batch_level(const BatchSys<typename C::T> *__restrict__ sys,
                                                                       const BatchPart *__restrict__ parts,
                                                                       int nparts) {
    extern __shared__ __align__(16) char sm[];
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const RefArgs<typename C::T> a = sys[P.sys].ref;
    refactor_block<C>(blockIdx.x - P.blk0, P.nblk, P.item0, a, P.nwide, P.small0, P.nsmall, P.c,
                      FuseArgs<typename C::T>{}, sm);
}

// A level whose wide items are all medium ones of wavefront levels, in every handle: as
// k_refactor_wave, with shares
template <class T, bool kMany>
__global__ __launch_bounds__(256, 3) void k_batch_wave(const BatchSys<T> *__restrict__ sys,
                                                       const BatchPart *__restrict__ parts, int nparts) {
    __shared__ __align__(16) char sm[sizeof(WaveLds<T>) * 4];
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const RefArgs<T> a = sys[P.sys].ref;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nmb = (P.nwide + 3) / 4, nsb = (P.nsmall + kBlock / 16 - 1) / (kBlock / 16);
    const int b = blockIdx.x - P.blk0;
    if (b < nmb) {
        const int i = b * 4 + wv;
        if (i < P.nwide) wave_item<T>(P.item0 + i, a, reinterpret_cast<WaveLds<T> *>(sm)[wv], i);
    } else if (b < nmb + nsb) {
        small_group<T, true, kMany>(P.small0, P.nsmall, a, (b - nmb) * (kBlock / 16) + (threadIdx.x >> 4),
                                    (b - nmb) * 4 + wv);
    } else {
        copy_block(a, P.c, b - nmb - nsb, P.nblk - nmb - nsb, kBlock);
    }
}

// the solve's set-up of every handle (grid y), unknowns marked unset; the first clears the tickets
template <class T>
__global__ __launch_bounds__(256) void k_batch_reset(const BatchSys<T> *__restrict__ sys,
                                                     const BatchPtrs *__restrict__ ptrs, int *tick) {
    const BatchSys<T> &S = sys[blockIdx.y];
    double *bp = const_cast<double *>(S.l.bp);
    solve_reset_body(blockIdx.x * blockDim.x + threadIdx.x, S.n, ptrs[blockIdx.y].b, S.r, S.P, bp, S.l.y, S.l.xt,
                     S.l.psum, S.l.usum, 1, blockIdx.y ? 0 : 2, tick);
}

// One triangle of every handle: blocks take entries of order (handle, item) by ticket
template <bool kFwd, class T>
__global__ __launch_bounds__(kPersThreads) void k_batch_solve(const BatchSys<T> *__restrict__ sys,
                                                              const BatchPtrs *__restrict__ ptrs,
                                                              const int2 *__restrict__ order, int total, int *tick) {
    __shared__ SolveLds L;
    if (threadIdx.x == kBlock) L.next[0] = atomicAdd(tick, 1);
    __syncthreads();
    int cur = L.next[0];
    for (int par = 1; cur < total; par ^= 1) {
        int nt = 0;
        if (threadIdx.x == kBlock) nt = atomicAdd(tick, 1);
        const int2 o = order[__builtin_amdgcn_readfirstlane(cur)];
        const int q = __builtin_amdgcn_readfirstlane(o.x);
        SolveArgs<T> a = kFwd ? sys[q].l : sys[q].u;
        if constexpr (!kFwd) a.x = ptrs[q].x;
        solve_item<kFwd>(a, __builtin_amdgcn_readfirstlane(o.y), L);
        if (threadIdx.x == kBlock) L.next[par] = nt;
        __syncthreads();
        cur = L.next[par];
    }
}

// norms of every handle's residual (grid y; a handle's own number of blocks)
template <class T>
__global__ __launch_bounds__(256) void k_batch_residual(const BatchSys<T> *__restrict__ sys,
                                                        const BatchPtrs *__restrict__ ptrs) {
    const BatchSys<T> &S = sys[blockIdx.y];
    if ((int)blockIdx.x >= S.nb_norm) return;
    const BatchPtrs p = ptrs[blockIdx.y];
    residual_body(blockIdx.x, S.nb_norm, S.n, S.a_rowptr, S.a_colind, p.v, p.x, p.b, nullptr, S.rpart, nullptr);
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_result(const BatchSys<T> *__restrict__ sys, int norms,
                                                      BatchResult *__restrict__ out) {
    const BatchSys<T> &S = sys[blockIdx.x];
    if (norms) max_parts_body(S.nb_norm, 3, S.rpart, &out[blockIdx.x].rn.rnorm);
    if (threadIdx.x == 0) out[blockIdx.x].st = *S.ref.st;
}

// the copy after the last level and the replaced-pivot sums
template <class T>
__global__ void k_batch_copy(const BatchSys<T> *__restrict__ sys, const BatchPart *__restrict__ parts, int nparts) {
    const BatchPart P = parts[find_part(parts, nparts, blockIdx.x)];
    const BatchSys<T> &S = sys[P.sys];
    copy_ranges(S.ref.copy_k, S.ref.copy_src, S.ref.lu, S.ref.lucsr, S.rest, blockIdx.x - P.blk0, P.nblk,
                blockDim.x);
}

template <class T>
__global__ __launch_bounds__(256) void k_batch_counts(const BatchSys<T> *__restrict__ sys) {
    sum_counts_body(sys[blockIdx.x].ref.pcount, &sys[blockIdx.x].ref.st->perturbed);
}

}  // namespace kkt

// worker threads (and streams) of kkt_batch_refine
constexpr int kBatchRefineThreads = 8;

struct kkt_batch {
    std::vector<kkt_handle *> hs;
    std::vector<char *> ws;        // each handle's workspace and schedule when the batch was made:
    std::vector<uint64_t> sch_id;  // its device tables point into that workspace, laid out for that schedule
    int device = -1;
    bool fp32 = false;
    char *dmem = nullptr;          // device: systems, shares, value-pointer table
    void *d_sys = nullptr;
    const double **d_vals = nullptr;
    const double **h_vals = nullptr;   // pinned staging of the value pointers
    hipEvent_t vals_done = nullptr;    // the last upload of h_vals has been read
    // launches of a step: kind (0 clear, 1 rows, 2 cols, 3 norms, 5 level,
    // 6 copy, 7 counts, 8 wavefront level, 9 the same with many narrow items), grid, first share,
    // shares
    struct Launch {
        int kind, grid, p0, np;
    };
    std::vector<Launch> launches;
    BatchPart *d_parts = nullptr;
    hipStream_t cap = nullptr;
    hipGraphExec_t graph = nullptr;
    hipEvent_t graph_done = nullptr;
    bool graph_failed = false;
    // concurrent refinement: one stream per worker thread, and an event that orders them
    // after the caller's stream
    std::vector<hipStream_t> rstreams;
    hipEvent_t ready = nullptr;
    // merged first solves of the refinement: items of all handles in level order
    int nl = 0, nu = 0, grid_l = 1, grid_u = 1, nmax = 0, nbmax = 0;
    int2 *d_lord = nullptr, *d_uord = nullptr;
    int *d_tick = nullptr;
    BatchPtrs *d_ptrs = nullptr, *h_ptrs = nullptr;     // device table, its pinned staging
    BatchResult *d_res = nullptr, *h_res = nullptr;
};

namespace {

template <class T>
BatchSys<T> batch_sys(const kkt_handle *h) {
    const Dev &d = h->d;
    const Schedule &g = h->sch;
    BatchSys<T> b{};
    b.ref = RefArgs<T>{d.ldiag, d.itemrec, d.pair8, d.f_rel, static_cast<T *>(d.lu), d.st, d.pcount,
                       std::is_same<T, float>::value ? h->opts.tiny_pivot_fp32 : h->opts.tiny_pivot,
                       h->opts.dense_mfma != 0, d.copy_k, d.copy_src, static_cast<T *>(d.lucsr),
                       d.pan_start, d.pan_r};
    b.a_rowptr = d.a_rowptr;
    b.a_colind = d.a_colind;
    b.colptr = d.colptr;
    b.Q = d.Q;
    b.lu_src = d.lu_src;
    b.r = d.r;
    b.c = d.c;
    b.er = d.er;
    b.ec = d.ec;
    b.n = h->sym.n;
    b.eq = h->opts.equilibrate != 0;
    b.nb_norm = norm_blocks(h->sym.n);
    b.rest = copy_rest(g, copy_carriers(g));
    b.l = SolveArgs<T>{d.l_item4, d.l_rows4, d.rinfo4, d.csr_col, d.Q, static_cast<const T *>(d.lucsr), d.c, d.bp,
                       d.y, d.xt, nullptr, d.call, d.psum, d.usum, &d.st->abort, nullptr, nullptr, 0, b.n, 1};
    b.u = b.l;
    b.u.item = d.u_item4;
    b.u.rows = d.u_rows4;
    b.u.rinfo = d.urinfo4;
    b.P = d.P;
    b.rpart = d.part;
    return b;
}

template <class T>
int batch_build(kkt_batch *b, std::vector<BatchPart> &parts, std::vector<char> &sysbytes) {
    using Big = BigCfg<T>;
    const int count = (int)b->hs.size();
    std::vector<BatchSys<T>> sys(count);
    for (int i = 0; i < count; ++i) sys[i] = batch_sys<T>(b->hs[i]);
    sysbytes.resize(sizeof(BatchSys<T>) * count);
    std::memcpy(sysbytes.data(), sys.data(), sysbytes.size());
    auto add = [&](int kind, const std::vector<BatchPart> &ps) {
        int grid = 0;
        for (const auto &p : ps) grid = std::max(grid, p.blk0 + p.nblk);
        if (grid == 0 && kind != 0 && kind != 7) return;
        b->launches.push_back({kind, kind == 0 || kind == 7 ? count : grid, (int)parts.size(),
                               (int)ps.size()});
        parts.insert(parts.end(), ps.begin(), ps.end());
    };
    auto shares = [&](auto nblk_of) {
        std::vector<BatchPart> ps;
        int blk = 0;
        for (int i = 0; i < count; ++i) {
            BatchPart p{};
            p.sys = i;
            p.blk0 = blk;
            p.nblk = nblk_of(i, p);
            if (p.nblk > 0) {
                ps.push_back(p);
                blk += p.nblk;
            }
        }
        return ps;
    };
    add(0, {});
    add(1, shares([&](int i, BatchPart &) { return row_blocks(sys[i].n); }));
    add(2, shares([&](int i, BatchPart &) { return col_blocks(sys[i].n); }));
    add(3, shares([&](int i, BatchPart &) { return sum_blocks(sys[i].n); }));
    int nlev = 0;
    for (auto *h : b->hs) nlev = std::max(nlev, (int)h->sch.f_lvl.size() - 1);
    for (int l = 0; l < nlev; ++l) {
        // on wavefronts where every handle's level allows it
        bool wave = true;
        int64_t narrow = 0;
        for (auto *h : b->hs) {
            const Schedule &g = h->sch;
            if (l + 1 >= (int)g.f_lvl.size()) continue;
            wave &= h->opts.dense_mfma != 0 && (g.f_wave[l] || g.f_nlarge[l] == 0);
            narrow += g.f_lvl[l + 1] - g.f_lvl[l] - g.f_nlarge[l];
        }
        const int threads = wave ? kBlock : Big::kThreads;
        add(!wave ? 5 : narrow >= kManyItems ? 9 : 8, shares([&](int i, BatchPart &p) {
            const kkt_handle *h = b->hs[i];
            const Schedule &g = h->sch;
            if (l + 1 >= (int)g.f_lvl.size()) return 0;
            const int i0 = g.f_lvl[l], nw = g.f_nlarge[l], ns = g.f_lvl[l + 1] - i0 - nw;
            const int ncopy = copy_carriers(g), cc = l - g.copy_lvl;
            const bool copy = cc >= 0 && cc < ncopy && nw > 0;
            p.item0 = i0;
            p.nwide = nw;
            p.small0 = i0 + nw;
            p.nsmall = ns;
            p.c = copy ? copy_chunk(g, cc, ncopy) : CopyRanges{0, 0, 0, 0};
            const int cb = copy_count(p.c) > 0 ? h->ncu : 0;
            return (wave ? (int)blocks_for(nw, 4) : nw) + (int)blocks_for(ns, threads / 16) + cb;
        }));
    }
    add(6, shares([&](int i, BatchPart &) { return (int)blocks_for(copy_count(sys[i].rest), 256); }));
    add(7, {});
    return KKT_OK;
}

template <class T>
int batch_enqueue(kkt_batch *b, hipStream_t s) {
    using Big = BigCfg<T>;
    const auto *sys = static_cast<const BatchSys<T> *>(b->d_sys);
    for (const auto &L : b->launches) {
        const BatchPart *p = b->d_parts + L.p0;
        switch (L.kind) {
            case 0: k_batch_clear<T><<<L.grid, 256, 0, s>>>(sys); break;
            case 1: k_batch_rows<T><<<L.grid, 256, 0, s>>>(sys, p, L.np, b->d_vals); break;
            case 2: k_batch_cols<T><<<L.grid, 256, 0, s>>>(sys, p, L.np, b->d_vals); break;
            case 3: k_batch_rowsums<T><<<L.grid, 256, 0, s>>>(sys, p, L.np, b->d_vals); break;
            case 5: k_batch_level<Big><<<L.grid, Big::kThreads, Big::kLds, s>>>(sys, p, L.np); break;
            case 6: k_batch_copy<T><<<L.grid, 256, 0, s>>>(sys, p, L.np); break;
            case 7: k_batch_counts<T><<<L.grid, 256, 0, s>>>(sys); break;
            case 8: k_batch_wave<T, false><<<L.grid, kBlock, 0, s>>>(sys, p, L.np); break;
            case 9: k_batch_wave<T, true><<<L.grid, kBlock, 0, s>>>(sys, p, L.np); break;
        }
    }
    HIPCHK(hipGetLastError());
    return KKT_OK;
}

int batch_enqueue_any(kkt_batch *b, hipStream_t s) {
    return b->fp32 ? batch_enqueue<float>(b, s) : batch_enqueue<double>(b, s);
}

void batch_free(kkt_batch *b) {
    if (b->device >= 0) {
        DeviceGuard g(b->device);
        if (b->graph_done) (void)hipEventSynchronize(b->graph_done);
        if (b->vals_done) (void)hipEventSynchronize(b->vals_done);
        if (b->cap) (void)hipStreamSynchronize(b->cap);
        if (b->graph) (void)hipGraphExecDestroy(b->graph);
        if (b->cap) (void)hipStreamDestroy(b->cap);
        if (b->graph_done) (void)hipEventDestroy(b->graph_done);
        for (hipStream_t st : b->rstreams) (void)hipStreamDestroy(st);
        if (b->ready) (void)hipEventDestroy(b->ready);
        if (b->vals_done) (void)hipEventDestroy(b->vals_done);
        if (b->dmem) (void)hipFree(b->dmem);
        if (b->h_vals) (void)hipHostFree(b->h_vals);
        if (b->h_ptrs) (void)hipHostFree(b->h_ptrs);
        if (b->h_res) (void)hipHostFree(b->h_res);
    }
    delete b;
}

// the batch's tables still describe handle i: not unbound, bound elsewhere or given another
// schedule since (a rebuilt schedule lays the same workspace address out anew)
bool batch_tables_hold(const kkt_batch *b, int i) {
    const kkt_handle *h = b->hs[i];
    return h->bound && h->ws == b->ws[i] && h->sch_id == b->sch_id[i];
}

// whether na doubles at a and nb doubles at b share memory
bool arrays_overlap(const double *a, int64_t na, const double *b, int64_t nb) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return p < q + sizeof(double) * nb && q < p + sizeof(double) * na;
}

// (handle, item) of every handle's solve items, level by level
void batch_order(const kkt_batch *b, bool fwd, std::vector<int2> &ord) {
    size_t nlev = 0;
    for (auto *h : b->hs) nlev = std::max(nlev, (fwd ? h->sch.l_lvl : h->sch.u_lvl).size() - 1);
    for (size_t l = 0; l < nlev; ++l)
        for (size_t q = 0; q < b->hs.size(); ++q) {
            const std::vector<int32_t> &lvl = fwd ? b->hs[q]->sch.l_lvl : b->hs[q]->sch.u_lvl;
            if (l + 1 >= lvl.size()) continue;
            for (int32_t it = lvl[l]; it < lvl[l + 1]; ++it) ord.push_back(int2{(int)q, it});
        }
}

template <class T>
int batch_first_solves_t(kkt_batch *b, hipStream_t s) {
    const auto *sys = static_cast<const BatchSys<T> *>(b->d_sys);
    const unsigned cnt = (unsigned)b->hs.size();
    k_batch_reset<T><<<dim3(blocks_for(b->nmax, 256), cnt), 256, 0, s>>>(sys, b->d_ptrs, b->d_tick);
    k_batch_solve<true, T><<<std::min(b->nl, b->grid_l), kPersThreads, 0, s>>>(sys, b->d_ptrs, b->d_lord, b->nl,
                                                                              b->d_tick);
    k_batch_solve<false, T><<<std::min(b->nu, b->grid_u), kPersThreads, 0, s>>>(sys, b->d_ptrs, b->d_uord, b->nu,
                                                                               b->d_tick + 1);
    k_batch_residual<T><<<dim3(b->nbmax, cnt), 256, 0, s>>>(sys, b->d_ptrs);
    k_batch_result<T><<<cnt, 256, 0, s>>>(sys, 1, b->d_res);
    HIPCHK(hipGetLastError());
    return KKT_OK;
}

// the handles' status blocks (and residual norms) to h_res; waits
template <class T>
int batch_status_t(kkt_batch *b, hipStream_t s) {
    k_batch_result<T><<<(unsigned)b->hs.size(), 256, 0, s>>>(static_cast<const BatchSys<T> *>(b->d_sys), 0, b->d_res);
    HIPCHK(hipGetLastError());
    return KKT_OK;
}
int batch_read(kkt_batch *b, hipStream_t s) {
    HIPCHK(hipMemcpyAsync(b->h_res, b->d_res, sizeof(BatchResult) * b->hs.size(), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return KKT_OK;
}

}  // namespace

extern "C" {

int kkt_batch_create(kkt_handle *const *handles, int32_t count, kkt_batch **out) {
    if (!out) return KKT_ERR_ARG;
    *out = nullptr;
    if (!handles || count < 1) return KKT_ERR_ARG;
    for (int32_t i = 0; i < count; ++i) {
        if (!handles[i]) return KKT_ERR_ARG;
        for (int32_t j = 0; j < i; ++j)
            if (handles[j] == handles[i]) return KKT_ERR_ARG;   // one workspace, one slot
        if (!handles[i]->bound) return KKT_ERR_STATE;
        if (handles[i]->device != handles[0]->device ||
            handles[i]->opts.factor_precision != handles[0]->opts.factor_precision)
            return KKT_ERR_ARG;
    }
    kkt_batch *b = new (std::nothrow) kkt_batch;
    if (!b) return KKT_ERR_NOMEM;
    b->hs.assign(handles, handles + count);
    for (auto *h : b->hs) {
        b->ws.push_back(h->ws);
        b->sch_id.push_back(h->sch_id);
    }
    b->device = handles[0]->device;
    b->fp32 = handles[0]->opts.factor_precision == KKT_FP32;
    DeviceGuard dg(b->device);
    if (!dg.ok) { batch_free(b); return KKT_ERR_DEVICE; }
    std::vector<BatchPart> parts;
    std::vector<char> sysbytes;
    int rc;
    try {
        rc = b->fp32 ? batch_build<float>(b, parts, sysbytes) : batch_build<double>(b, parts, sysbytes);
    } catch (const std::bad_alloc &) {
        rc = KKT_ERR_NOMEM;
    }
    if (rc) { batch_free(b); return rc; }
    const size_t off_parts = (sysbytes.size() + 255) & ~size_t(255);
    const size_t off_vals = (off_parts + parts.size() * sizeof(BatchPart) + 255) & ~size_t(255);
    std::vector<int2> lord, uord;
    try {
        batch_order(b, true, lord);
        batch_order(b, false, uord);
    } catch (const std::bad_alloc &) {
        batch_free(b);
        return KKT_ERR_NOMEM;
    }
    auto after = [](size_t off, size_t bytes) { return (off + bytes + 255) & ~size_t(255); };
    const size_t off_ptrs = after(off_vals, sizeof(double *) * count);
    const size_t off_res = after(off_ptrs, sizeof(BatchPtrs) * count);
    const size_t off_tick = after(off_res, sizeof(BatchResult) * count);
    const size_t off_lord = after(off_tick, 2 * sizeof(int));
    const size_t off_uord = after(off_lord, sizeof(int2) * lord.size());
    const size_t total = after(off_uord, sizeof(int2) * uord.size());
    if (hipMalloc(&b->dmem, total) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void **>(&b->h_ptrs), sizeof(BatchPtrs) * count) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void **>(&b->h_res), sizeof(BatchResult) * count) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void **>(&b->h_vals), sizeof(double *) * count) != hipSuccess ||
        hipEventCreateWithFlags(&b->vals_done, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->graph_done, hipEventDisableTiming) != hipSuccess ||
        hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->ready, hipEventDisableTiming) != hipSuccess) {
        batch_free(b);
        return KKT_ERR_DEVICE;
    }
    for (int i = 0; i < std::min(count, kBatchRefineThreads); ++i) {
        hipStream_t st = nullptr;
        if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
            batch_free(b);
            return KKT_ERR_DEVICE;
        }
        b->rstreams.push_back(st);
    }
    {
        const hipError_t e = b->fp32 ? hipFuncSetAttribute(reinterpret_cast<const void *>(&k_batch_level<BigCfg<float>>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                                           BigCfg<float>::kLds)
                                     : hipFuncSetAttribute(reinterpret_cast<const void *>(&k_batch_level<BigCfg<double>>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                                           BigCfg<double>::kLds);
        if (e != hipSuccess) {
            batch_free(b);
            return KKT_ERR_DEVICE;
        }
    }
    b->d_sys = b->dmem;
    b->d_parts = reinterpret_cast<BatchPart *>(b->dmem + off_parts);
    b->d_vals = reinterpret_cast<const double **>(b->dmem + off_vals);
    b->d_ptrs = reinterpret_cast<BatchPtrs *>(b->dmem + off_ptrs);
    b->d_res = reinterpret_cast<BatchResult *>(b->dmem + off_res);
    b->d_tick = reinterpret_cast<int *>(b->dmem + off_tick);
    b->d_lord = reinterpret_cast<int2 *>(b->dmem + off_lord);
    b->d_uord = reinterpret_cast<int2 *>(b->dmem + off_uord);
    b->nl = (int)lord.size();
    b->nu = (int)uord.size();
    for (auto *h : b->hs) {
        b->nmax = std::max(b->nmax, h->sym.n);
        b->nbmax = std::max(b->nbmax, norm_blocks(h->sym.n));
    }
    {
        int bl = 0, bu = 0;
        auto occ = [&](auto tag) {
            using T = decltype(tag);
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                       &bl, reinterpret_cast<const void *>(&k_batch_solve<true, T>), kPersThreads, 0) == hipSuccess &&
                   hipOccupancyMaxActiveBlocksPerMultiprocessor(
                       &bu, reinterpret_cast<const void *>(&k_batch_solve<false, T>), kPersThreads, 0) == hipSuccess;
        };
        if (!(b->fp32 ? occ(float{}) : occ(double{}))) {
            batch_free(b);
            return KKT_ERR_DEVICE;
        }
        b->grid_l = std::max(1, bl) * b->hs[0]->ncu;
        b->grid_u = std::max(1, bu) * b->hs[0]->ncu;
    }
    if ((!lord.empty() && hipMemcpy(b->d_lord, lord.data(), sizeof(int2) * lord.size(), hipMemcpyHostToDevice) != hipSuccess) ||
        (!uord.empty() && hipMemcpy(b->d_uord, uord.data(), sizeof(int2) * uord.size(), hipMemcpyHostToDevice) != hipSuccess)) {
        batch_free(b);
        return KKT_ERR_DEVICE;
    }
    if (hipMemcpy(b->d_sys, sysbytes.data(), sysbytes.size(), hipMemcpyHostToDevice) != hipSuccess ||
        (!parts.empty() && hipMemcpy(b->d_parts, parts.data(), parts.size() * sizeof(BatchPart),
                                     hipMemcpyHostToDevice) != hipSuccess) ||
        hipEventRecord(b->vals_done, nullptr) != hipSuccess) {
        batch_free(b);
        return KKT_ERR_DEVICE;
    }
    *out = b;
    return KKT_OK;
}

int kkt_batch_refactor(kkt_batch *b, const double *const *d_values, hipStream_t stream) {
    if (!b || !d_values) return KKT_ERR_ARG;
    const int count = (int)b->hs.size();
    for (int i = 0; i < count; ++i) {
        if (!d_values[i]) return KKT_ERR_ARG;
        if (!batch_tables_hold(b, i)) return KKT_ERR_STATE;
    }
    DeviceGuard dg(b->device);
    if (!dg.ok) return KKT_ERR_DEVICE;
    // the pinned staging of the value pointers is rewritten once its last upload was read
    HIPCHK(hipEventSynchronize(b->vals_done));
    for (int i = 0; i < count; ++i) b->h_vals[i] = d_values[i];
    HIPCHK(hipMemcpyAsync(b->d_vals, b->h_vals, sizeof(double *) * count, hipMemcpyHostToDevice, stream));
    HIPCHK(hipEventRecord(b->vals_done, stream));
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    HIPCHK(hipStreamIsCapturing(stream, &cs));
    int rc = KKT_OK;
    if (!b->graph && !b->graph_failed && cs == hipStreamCaptureStatusNone) {
        hipGraph_t graph = nullptr;
        if (hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal) == hipSuccess) {
            const int erc = batch_enqueue_any(b, b->cap);
            const hipError_t e = hipStreamEndCapture(b->cap, &graph);
            if (erc || e != hipSuccess || !graph || hipGraphInstantiate(&b->graph, graph, nullptr, nullptr, 0) != hipSuccess) {
                (void)hipGetLastError();
                b->graph = nullptr;
                b->graph_failed = true;
            }
            if (graph) (void)hipGraphDestroy(graph);
        } else {
            (void)hipGetLastError();
            b->graph_failed = true;
        }
    }
    if (b->graph && cs == hipStreamCaptureStatusNone) {
        HIPCHK(hipGraphLaunch(b->graph, stream));
        HIPCHK(hipEventRecord(b->graph_done, stream));
    } else {
        rc = batch_enqueue_any(b, stream);
        if (rc) return rc;
    }
    for (int i = 0; i < count; ++i) {
        b->hs[i]->d_values = d_values[i];
        b->hs[i]->factored = true;
    }
    return KKT_OK;
}

int kkt_batch_refine(kkt_batch *b, const double *const *d_b, double *const *d_x, kkt_info *info,
                     hipStream_t stream) {
    if (!b || !d_b || !d_x) return KKT_ERR_ARG;
    const int count = (int)b->hs.size();
    for (int i = 0; i < count; ++i)
        if (!d_b[i] || !d_x[i]) return KKT_ERR_ARG;
    DeviceGuard dg(b->device);
    if (!dg.ok) return KKT_ERR_DEVICE;
    std::vector<int> rcs(count, KKT_OK);
    std::vector<kkt_info> infs(count);
    // the first solves of all handles together, where every handle can take part: refactored, as
    // the batch's tables describe it, not profiled, its solution over no right-hand side
    // and no other solution, its factors sound
    bool merged = true;
    for (int i = 0; i < count; ++i) {
        const kkt_handle *h = b->hs[i];
        merged &= batch_tables_hold(b, i) && h->factored && !h->prof && h->opts.persistent_solve != 0;
        for (int j = 0; j < count && merged; ++j) {
            const int n = h->sym.n, nj = b->hs[j]->sym.n;
            merged &= !arrays_overlap(d_b[i], n, d_x[j], nj) && (i == j || !arrays_overlap(d_x[i], n, d_x[j], nj));
        }
    }
    std::vector<char> solved(count, 0);
    if (merged) {
        int rc = b->fp32 ? batch_status_t<float>(b, stream) : batch_status_t<double>(b, stream);
        if (!rc) rc = batch_read(b, stream);
        if (rc) return rc;
        for (int i = 0; i < count; ++i)
            merged &= !(b->h_res[i].st.flags & (kFlagInternal | kFlagNonfinite)) && !b->h_res[i].st.abort;
    }
    if (merged) {
        // the staging was last read before the wait above
        for (int i = 0; i < count; ++i) b->h_ptrs[i] = BatchPtrs{b->hs[i]->d_values, d_b[i], d_x[i]};
        HIPCHK(hipMemcpyAsync(b->d_ptrs, b->h_ptrs, sizeof(BatchPtrs) * count, hipMemcpyHostToDevice, stream));
        int rc = b->fp32 ? batch_first_solves_t<float>(b, stream) : batch_first_solves_t<double>(b, stream);
        if (!rc) rc = batch_read(b, stream);
        if (rc) return rc;
        for (int i = 0; i < count; ++i) {
            const int rc1 = first_info(b->h_res[i].st, b->h_res[i].rn, b->hs[i]->opts.berr_tol, &infs[i]);
            rcs[i] = std::min(rc1, KKT_OK);
            solved[i] = rc1 == KKT_WARN_NOT_CONVERGED ? 1 : 2;   // 2: done
        }
    }
    // the rest by worker threads on streams that start after everything enqueued so far
    if (std::any_of(solved.begin(), solved.end(), [](char c) { return c != 2; })) {
        HIPCHK(hipEventRecord(b->ready, stream));
        for (hipStream_t st : b->rstreams) HIPCHK(hipStreamWaitEvent(st, b->ready, 0));
        std::atomic<int> next(0);
        auto work = [&](hipStream_t st) {
            (void)hipSetDevice(b->device);
            for (int i; (i = next.fetch_add(1)) < count;) {
                if (solved[i] == 2) continue;
                const int64_t pert = infs[i].perturbed_pivots;
                if (solved[i] == 0) {
                    rcs[i] = kkt_refine(b->hs[i], d_b[i], d_x[i], 1, b->hs[i]->sym.n, &infs[i], st);
                } else {
                    rcs[i] = fgmres_column(b->hs[i], d_b[i], d_x[i], &infs[i], st, kSolved);
                    infs[i].perturbed_pivots = pert;
                }
                if (rcs[i] < 0) info_error(rcs[i], pert, &infs[i]);
            }
        };
        std::vector<std::thread> pool;
        try {
            for (size_t t = 1; t < b->rstreams.size(); ++t) pool.emplace_back(work, b->rstreams[t]);
        } catch (...) {
            // fewer threads: the remaining handles go to the ones that started
        }
        work(b->rstreams[0]);
        for (auto &t : pool) t.join();
    }
    int worst = KKT_OK;
    for (int i = 0; i < count; ++i) {
        if (info) info[i] = infs[i];
        if (rcs[i] < 0 && worst >= 0) worst = rcs[i];
        else if (worst >= 0) worst = std::max(worst, rcs[i]);
    }
    return worst;
}

void kkt_batch_destroy(kkt_batch *b) {
    if (b) batch_free(b);
}

}  // extern "C"
